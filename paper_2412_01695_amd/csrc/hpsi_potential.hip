// What the H|psi> kernels read of the potential besides V on its own mesh.
//
// The local term couples plane waves of one k-point only, so of the transform
// V~ of V(r) (Eq. fwFFT, with 1/N_r) it reads V~[d mod N] at the Miller
// differences |d_a| <= W_a - 1 of the window W1 x W2 x W3.  The same values put
// on any mesh of at least 2 W_a - 1 points per axis give the same operator: the
// mesh of a density (twice the wave-function sphere and more) is larger than
// that, and H|psi> runs on the smallest compiled mesh that is enough: for 36^3
// with a window of 11 that is 24^3, 3.4 times fewer points (1728 k x 24 bands:
// 4.11 -> 1.86 ms in FP64, 1.82 -> 0.90 ms in complex64), for 30^3 and 24^3 with
// a window of 10 it is 20^3 (2048 k x 16 bands at 30^3 in complex64: 0.87 -> 0.46
// ms; 512 k x 20 bands at 24^3 in FP64: 0.38 -> 0.32 ms).  Fewer points are less
// work in every pass: over meshes of 15^3 to 36^3, 4 to 32 projectors and both
// precisions launches of 300 to 1000 k took 0.30 to 1.02 times as long as on the
// context's mesh with shapes tuned for them (launches of few rows need shapes of their
// own, launch_one in hpsi_kernel.hpp).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "internal.hpp"

namespace mkpw {

namespace {

typedef cplx<double> cd;

// One axis of V~ over the box of differences: in is [outer][n][inner] (real or
// complex), out [outer][2 w - 1][inner],
// out(d) = sum_l in(l) exp(-2 pi i d l / n), d = -(w - 1) .. w - 1.
template <class In>
__global__ __launch_bounds__(256) void to_box_kernel(const In* __restrict__ in, cd* __restrict__ out, int outer, int n,
                                                     int inner, int w) {
  const int dw = 2 * w - 1;
  const long total = (long)outer * dw * inner;
  for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < total; e += (long)gridDim.x * 256) {
    const int i = (int)(e % inner);
    const long t = e / inner;
    const int d = ((int)(t % dw) - (w - 1) + n * w) % n;
    const long o = t / dw;
    double sr = 0.0, si = 0.0;
    int ph = 0;  // d l mod n
    for (int l = 0; l < n; ++l) {
      double sn, cs;
      sincospi(2.0 * ph / n, &sn, &cs);
      if constexpr (sizeof(In) == sizeof(double)) {
        const double v = in[(o * n + l) * inner + i];
        sr += v * cs;
        si -= v * sn;
      } else {
        const cd v = in[(o * n + l) * inner + i];
        sr += v.x * cs + v.y * sn;
        si += v.y * cs - v.x * sn;
      }
      ph += d;
      if (ph >= n) ph -= n;
    }
    out[e] = {sr, si};
  }
}

// One axis of the way back onto a mesh of n points: in is [outer][2 w - 1][inner],
// out(l) = sum_d in(d) exp(2 pi i d l / n), [outer][n][inner].
__global__ __launch_bounds__(256) void from_box_kernel(const cd* __restrict__ in, cd* __restrict__ out, int outer,
                                                       int n, int inner, int w) {
  const int dw = 2 * w - 1;
  const long total = (long)outer * n * inner;
  for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < total; e += (long)gridDim.x * 256) {
    const int i = (int)(e % inner);
    const long t = e / inner;
    const int l = (int)(t % n);
    const long o = t / n;
    double sr = 0.0, si = 0.0;
    int ph = ((1 - w) * l % n + n) % n;  // d l mod n
    for (int d = 0; d < dw; ++d) {
      double sn, cs;
      sincospi(2.0 * ph / n, &sn, &cs);
      const cd v = in[(o * dw + d) * inner + i];
      sr += v.x * cs - v.y * sn;
      si += v.y * cs + v.x * sn;
      ph += l;
      if (ph >= n) ph -= n;
    }
    out[e] = {sr, si};
  }
}

// V / N_r on the mesh, in both precisions (V is real: V~(-d) = conj V~(d))
__global__ __launch_bounds__(256) void real_part_kernel(const cd* __restrict__ in, long n, double scale,
                                                        double* __restrict__ o64, float* __restrict__ o32) {
  for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < n; e += (long)gridDim.x * 256) {
    const double v = scale * in[e].x;
    o64[e] = v;
    o32[e] = (float)v;
  }
}

// the upper half of the box (linear offsets >= 0 from its centre; V~(-d) = conj
// V~(d)) in both precisions
__global__ __launch_bounds__(256) void half_box_kernel(const cd* __restrict__ in, long n, cd* __restrict__ o64,
                                                       cplx<float>* __restrict__ o32) {
  for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < n; e += (long)gridDim.x * 256) {
    o64[e] = in[e];
    o32[e] = {(float)in[e].x, (float)in[e].y};
  }
}

dim3 grid_of(long total) { return dim3((unsigned)std::min<long>(4096, (total + 255) / 256)); }

}  // namespace

void hpsi_potential_build(pw_ctx* c) {
  if (c->host_only || !c->have_k || !c->have_v) return;
  void** const kept[] = {&c->d_vk64, &c->d_vk32, &c->d_box64, &c->d_box32};
  auto drop = [&]() {
    for (void** p : kept) {
      dev_free(c, *p);
      *p = nullptr;
    }
    c->kmesh = c->kept_mesh = c->kept_half = 0;
  };
  c->stale_potential();
  const int n = c->fft[0];
  if (!hpsi_supported(c->fft[0], c->fft[1], c->fft[2])) return drop();
  const int w[3] = {c->wx, c->wy, c->wz};
  int m = hpsi_mesh_at_least(2 * std::max(w[0], std::max(w[1], w[2])) - 1);
  if (m >= n) m = 0;
  const long half = hpsi_dense_box(c);
  // (a new V on the same k-list is put in the same arrays)
  if (m != c->kept_mesh || half != c->kept_half) drop();
  if (m == 0 && half == 0) return;
  const long d1 = 2 * w[0] - 1, d2 = 2 * w[1] - 1, d3 = 2 * w[2] - 1, nr = (long)m * m * m;
  // two work arrays for the passes; without memory for them or for what is kept
  // the context has its own mesh alone
  const std::string err = c->err;
  const long most = std::max({d1 * n * n, d1 * d2 * n, d1 * d2 * d3, nr});
  void *a = nullptr, *b = nullptr;
  auto get = [&](long bytes, void** p) { return *p || dev_alloc(c, (size_t)bytes, p, true) == PW_OK; };
  bool ok = get(sizeof(cd) * most, &a) && get(sizeof(cd) * most, &b) && get(sizeof(double) * nr, &c->d_vk64) &&
            get(sizeof(float) * nr, &c->d_vk32) && get(sizeof(cd) * half, &c->d_box64) &&
            get(sizeof(cplx<float>) * half, &c->d_box32);
  if (ok) {
    cd *x = (cd*)a, *y = (cd*)b;
    const dim3 wg(256);
    hipStream_t st = c->stream;
    hipLaunchKernelGGL(to_box_kernel<double>, grid_of(d1 * n * n), wg, 0, st, c->d_v64, x, 1, n, n * n, w[0]);
    hipLaunchKernelGGL(to_box_kernel<cd>, grid_of(d1 * d2 * n), wg, 0, st, x, y, (int)d1, n, n, w[1]);
    hipLaunchKernelGGL(to_box_kernel<cd>, grid_of(d1 * d2 * d3), wg, 0, st, y, x, (int)(d1 * d2), n, 1, w[2]);
    if (half)
      hipLaunchKernelGGL(half_box_kernel, grid_of(half), wg, 0, st, x + d1 * d2 * d3 - half, half, (cd*)c->d_box64,
                         (cplx<float>*)c->d_box32);
    if (m) {
      hipLaunchKernelGGL(from_box_kernel, grid_of(d1 * d2 * m), wg, 0, st, x, y, (int)(d1 * d2), m, 1, w[2]);
      hipLaunchKernelGGL(from_box_kernel, grid_of(d1 * m * m), wg, 0, st, y, x, (int)d1, m, m, w[1]);
      hipLaunchKernelGGL(from_box_kernel, grid_of(nr), wg, 0, st, x, y, 1, m, m * m, w[0]);
      hipLaunchKernelGGL(real_part_kernel, grid_of(nr), wg, 0, st, y, nr, 1.0 / (double)nr, (double*)c->d_vk64,
                         (float*)c->d_vk32);
    }
    ok = hipGetLastError() == hipSuccess;
  }
  dev_free(c, a);
  dev_free(c, b);
  if (ok) {
    c->kmesh = c->kept_mesh = m;
    c->kept_half = (int)half;
  } else {
    drop();
    c->err = err;
  }
}

}  // namespace mkpw
