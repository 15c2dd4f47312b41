// Batched overlap operator (Sec. 2.2, Eqs. lambdah, delta_eq and finals):
//   lambda_q = <beta_q|psi>,  delta_p = sum_q q_pq lambda_q,
//   S psi    = psi + sum_p delta_p beta_p
// for every selected (k, band) row at once: two small products per k, on the
// matrix cores.  All rows of a k-point run on one XCD, so that the projector
// rows of a k are fetched from HBM into one L2 and served from there.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <string>

#include "internal.hpp"
#include "wave.hpp"  // dpp<>, wave_sum

namespace mkpw {

namespace {

constexpr int kSThreads = 256;
constexpr int kSMaxProj = 32;

// ------------------------------------------------------------------ on the matrix cores

// D (16 x 16) += A (16 x 4) B (4 x 16) per wave: lane l = 16 kq + l16 holds
// A[l16][kq] and B[kq][l16]; item r of the result is column l16 of row
// 4 r + kq (FP64) or 4 kq + r (FP32)
typedef double sf64x4 __attribute__((ext_vector_type(4)));
typedef float sf32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ sf64x4 smfma(double a, double b, sf64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ sf32x4 smfma(float a, float b, sf32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
template <class T>
struct SAcc {
  typedef sf64x4 type;
};
template <>
struct SAcc<float> {
  typedef sf32x4 type;
};
template <class T>
__device__ __forceinline__ int srow(int r, int kq) {
  return sizeof(T) == 8 ? 4 * r + kq : 4 * kq + r;
}

constexpr int kSBands = 8;      // rows of psi per workgroup
constexpr int kSMfmaProj = 16;  // one tile of projectors
constexpr int kSMfmaRow = 1024;  // longest rows

// One workgroup of four waves per (k, eight rows); the 16 columns of a tile are
// the real parts of the eight rows, then their imaginary parts.  A wave holds
// TW tiles of 16 plane waves of psi in registers, in the layout of a result
// tile, so the same registers are the B operand of lambda (an item r of a tile
// is a step of four plane waves) and the addend of sum_p beta_p delta_p.  Loads and stores take whole complex numbers: the
// lanes of the real columns those of an even item, the lanes of the imaginary
// columns those of the next, halves exchanged eight lanes apart.  The waves'
// lambdas meet in LDS, where delta is formed.
// Up to eight projectors the A rows of lambda hold Re beta, then Im beta (one
// product a step); P16 takes two.
// Bound by memory and the chain of a workgroup (load, lambda, barrier, delta, store):
// psi is read once, beta from the XCD's L2, the result written once.  512 k x 20 rows
// [305], 8 projectors, FP64, 120 MB, half a wave per row with lane sums / this: 56 / 36
// us called again and again on the same rows, which the last-level cache then holds; 60
// / 41 us (2.9 TB/s) on rows that come from HBM, twelve psi and results in turn.
template <class T, int TW, bool P16>
__global__ __launch_bounds__(kSThreads) __attribute__((amdgpu_waves_per_eu(TW <= 5 ? 4 : 1))) void spsi_mfma_kernel(
    const cplx<T>* psi, cplx<T>* out, long kstride, int nvec, const int* __restrict__ off,
    const int* __restrict__ cnt, const int* __restrict__ live, const int* __restrict__ npw_k, int npwx, int nproj,
    const cplx<T>* __restrict__ beta, const cplx<T>* __restrict__ q, const double* __restrict__ scale, double mult,
    int per_xcd, int ngroup, int groups_per_k) {
  typedef typename SAcc<T>::type acc_t;
  constexpr int NL = P16 ? 2 : 1, NJ = P16 ? 4 : 2;  // lambda tiles, steps over the projectors
  __shared__ T part[4][NL * 16][17];                 // each wave's lambda rows (Re beta, Im beta) by column
  __shared__ T lam[16][17], del[16][17];
  __shared__ cplx<T> qs[kSMfmaProj * kSMfmaProj];
  // workgroups are dealt to the 8 XCDs round-robin: the groups of one k go to
  // the same XCD
  const int grp = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (grp >= ngroup) return;
  const int k = grp / groups_per_k, r0 = (grp - k * groups_per_k) * kSBands;
  const int nrow = min(kSBands, (cnt ? cnt[k] : nvec) - r0);
  if (nrow <= 0) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l16 = lane & 15, kq = lane >> 4, b = l16 & 7, odd = l16 >> 3;
  const int task = k * nvec + r0 + (b < nrow ? b : 0);
  const bool act = b < nrow && !(live && !live[task]);
  if (__ballot(act) == 0) return;  // the same in every wave
  const int npw = npw_k[k];
  const long row = (long)k * kstride + (long)((off ? off[k] : 0) + r0 + (b < nrow ? b : 0)) * npwx;
  const cplx<T>* x = psi + row;
  cplx<T>* y = out + row;
  auto plane = [&](int i, int r) { return (wave + 4 * i) * 16 + srow<T>(r, kq); };
  if ((int)threadIdx.x < nproj * nproj) qs[threadIdx.x] = q[threadIdx.x];
  // psi: v[i][r] = this lane's part of plane wave plane(i, r) of row b
  acc_t v[TW];
  cplx<T> in[TW][2];
#pragma unroll
  for (int i = 0; i < TW; ++i) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int g = plane(i, 2 * h + odd);
      in[i][h] = x[act && g < npw ? g : 0];
    }
  }
#pragma unroll
  for (int i = 0; i < TW; ++i) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const bool ok = act && plane(i, 2 * h + odd) < npw;
      const T xr = ok ? in[i][h].x : T(0), xi = ok ? in[i][h].y : T(0);
      const T got = dpp<0x128>(odd ? xr : xi);  // row_ror:8
      v[i][2 * h] = odd ? got : xr;
      v[i][2 * h + 1] = odd ? xi : got;
    }
  }
  const cplx<T>* bk = beta + (long)k * nproj * npwx;
  if (nproj > 0) {
    // lambda_p = sum_G conj(beta_p(G)) psi(G)   (Eq. lambdah)
    acc_t la[NL][2];
#pragma unroll
    for (int n = 0; n < NL; ++n) la[n][0] = la[n][1] = acc_t{0, 0, 0, 0};
    const int pr = P16 ? l16 : l16 & 7;
    const cplx<T>* br = bk + (long)(pr < nproj ? pr : 0) * npwx;
#pragma unroll
    for (int i = 0; i < TW; ++i) {
      cplx<T> a[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int g = plane(i, r);
        a[r] = br[g < npw ? g : 0];
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const bool ok = plane(i, r) < npw;  // past the sphere psi is zero, and beta is taken as zero
        const T ax = ok ? a[r].x : T(0), ay = ok ? a[r].y : T(0);
        if constexpr (P16) {
          la[0][r & 1] = smfma(ax, v[i][r], la[0][r & 1]);
          la[NL - 1][r & 1] = smfma(ay, v[i][r], la[NL - 1][r & 1]);
        } else {
          la[0][r & 1] = smfma(odd ? ay : ax, v[i][r], la[0][r & 1]);
        }
      }
    }
    // beta for the last step, on its way while delta is formed
    cplx<T> bg[TW][NJ];
#pragma unroll
    for (int i = 0; i < TW; ++i) {
      const int g = (wave + 4 * i) * 16 + l16;
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        bg[i][j] = bk[(long)(4 * j + kq < nproj ? 4 * j + kq : 0) * npwx + (g < npw ? g : 0)];
    }
#pragma unroll
    for (int n = 0; n < NL; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) part[wave][16 * n + srow<T>(r, kq)][l16] = la[n][0][r] + la[n][1][r];
    __syncthreads();
    {
      // row p, column c of lambda: Re = Re beta . Re + Im beta . Im, Im = Re beta . Im - Im beta . Re
      const int p = threadIdx.x >> 4, c = threadIdx.x & 15, pi = P16 ? 16 + p : 8 + (p & 7);
      T s = T(0), t = T(0);
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        s += part[w][p][c];
        t += part[w][pi][c ^ 8];
      }
      lam[p][c] = c < 8 ? s + t : s - t;
    }
    __syncthreads();
    {
      // delta_p = sum_s q_ps lambda_s   (Eq. delta_eq)
      const int p = threadIdx.x >> 4, c = threadIdx.x & 15;
      T d = T(0);
      if (p < nproj) {
        for (int s = 0; s < nproj; ++s) {
          const cplx<T> qq = qs[p * nproj + s];
          const T own = lam[s][c], other = lam[s][c ^ 8];
          d += c < 8 ? qq.x * own - qq.y * other : qq.x * own + qq.y * other;
        }
      }
      del[p][c] = d;
    }
    __syncthreads();
    // S psi = psi + sum_p delta_p beta_p   (Eq. finals)
    T d1[NJ], d2[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      d1[j] = del[4 * j + kq][l16];
      d2[j] = odd ? del[4 * j + kq][l16 ^ 8] : -del[4 * j + kq][l16 ^ 8];
    }
#pragma unroll
    for (int i = 0; i < TW; ++i) {
      const int g = (wave + 4 * i) * 16 + l16;
      acc_t s = {0, 0, 0, 0};  // added to psi whole, so that psi's magnitude rounds once
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const bool ok = g < npw && 4 * j + kq < nproj;
        s = smfma(ok ? bg[i][j].x : T(0), d1[j], s);
        s = smfma(ok ? bg[i][j].y : T(0), d2[j], s);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) v[i][r] += s[r];
    }
  }
  const T f = scale ? T(mult * scale[task]) : T(1);
#pragma unroll
  for (int i = 0; i < TW; ++i) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const T got = dpp<0x128>(odd ? v[i][2 * h] : v[i][2 * h + 1]);
      const cplx<T> s = {odd ? got : v[i][2 * h], odd ? v[i][2 * h + 1] : got};
      const int g = plane(i, 2 * h + odd);
      if (!act || g >= npwx) continue;
      if (!scale) {
        y[g] = g < npw ? s : cplx<T>{T(0), T(0)};
      } else if (g < npw) {
        const cplx<T> o = y[g];
        y[g] = {o.x + f * s.x, o.y + f * s.y};
      }
    }
  }
}

// ------------------------------------------------------------------ on the vector units

// NP: nproj rounded up to a multiple of 8 (8 or 32), so that lambda and
// delta live in registers.  NPL > 0: each lane keeps its NPL plane waves
// (g = lane + 64 i) of psi in registers, loaded all at once, so the row is read
// from HBM once with every load in flight together; NPL = 0 (rows longer than
// 16 x 64) loops over the row and reads psi a second time for the output.
template <class T, int NP, int NPL>
__global__ __launch_bounds__(kSThreads) void spsi_kernel(const cplx<T>* psi, cplx<T>* out, long kstride, int nvec,
                                                         const int* __restrict__ off, const int* __restrict__ cnt,
                                                         const int* __restrict__ live, const int* __restrict__ npw_k,
                                                         int npwx, int nproj, const cplx<T>* __restrict__ beta,
                                                         const cplx<T>* __restrict__ q,
                                                         const double* __restrict__ scale, double mult, int per_xcd,
                                                         int ntask) {
  extern __shared__ char smem[];
  auto* qs = reinterpret_cast<cplx<T>*>(smem);  // q, nproj x nproj
  for (int e = threadIdx.x; e < nproj * nproj; e += kSThreads) qs[e] = q[e];
  __syncthreads();
  // workgroups are dealt to the 8 XCDs round-robin: consecutive rows (the
  // bands of one k) go to the same XCD
  const int bid = blockIdx.x;
  const int task = ((bid & 7) * per_xcd + (bid >> 3)) * (kSThreads / 64) + (int)(threadIdx.x >> 6);
  if (task >= ntask) return;
  const int k = task / nvec, r = task - k * nvec;
  if (r >= (cnt ? cnt[k] : nvec)) return;
  if (live && !live[task]) return;
  const int lane = threadIdx.x & 63;
  const long row = (long)k * kstride + (long)((off ? off[k] : 0) + r) * npwx;
  const cplx<T>* x = psi + row;
  cplx<T>* y = out + row;
  const int npw = npw_k[k];
  const cplx<T>* bk = beta + (long)k * nproj * npwx;
  constexpr int NC = NPL > 0 ? NPL : 1;
  cplx<T> xr[NC];
  if constexpr (NPL > 0) {
#pragma unroll
    for (int i = 0; i < NPL; ++i) {
      const int g = lane + 64 * i;
      xr[i] = g < npw ? x[g] : cplx<T>{T(0), T(0)};
    }
  }
  // lambda_p = sum_G conj(beta_p(G)) psi(G)   (Eq. lambdah), on every lane
  T lr[NP], li[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p) lr[p] = li[p] = T(0);
  auto accumulate = [&](int g, const cplx<T>& xv) {
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      if (p < nproj) {
        const cplx<T> bv = bk[(long)p * npwx + g];
        lr[p] += bv.x * xv.x + bv.y * xv.y;
        li[p] += bv.x * xv.y - bv.y * xv.x;
      }
    }
  };
  if constexpr (NPL > 0) {
#pragma unroll
    for (int i = 0; i < NPL; ++i)
      if (lane + 64 * i < npw) accumulate(lane + 64 * i, xr[i]);
  } else {
    for (int g = lane; g < npw; g += 64) accumulate(g, x[g]);
  }
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    if (p < nproj) {
      lr[p] = wave_sum(lr[p]);
      li[p] = wave_sum(li[p]);
    }
  }
  // delta_p = sum_s q_ps lambda_s   (Eq. delta_eq), on every lane
  T dr[NP], di[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    dr[p] = di[p] = T(0);
    if (p < nproj) {
#pragma unroll
      for (int s2 = 0; s2 < NP; ++s2) {
        if (s2 < nproj) {
          const cplx<T> qq = qs[p * nproj + s2];
          dr[p] += qq.x * lr[s2] - qq.y * li[s2];
          di[p] += qq.x * li[s2] + qq.y * lr[s2];
        }
      }
    }
  }
  // S psi = psi + sum_p delta_p beta_p   (Eq. finals)
  const T f = scale ? T(mult * scale[task]) : T(1);
  auto emit = [&](int g, cplx<T> v) {
    if (g >= npw) {
      if (!scale) y[g] = {T(0), T(0)};
      return;
    }
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      if (p < nproj) {
        const cplx<T> bv = bk[(long)p * npwx + g];
        v.x += dr[p] * bv.x - di[p] * bv.y;
        v.y += dr[p] * bv.y + di[p] * bv.x;
      }
    }
    if (scale) {
      const cplx<T> o = y[g];
      y[g] = {o.x + f * v.x, o.y + f * v.y};
    } else {
      y[g] = v;
    }
  };
  if constexpr (NPL > 0) {
#pragma unroll
    for (int i = 0; i < NPL; ++i)
      if (lane + 64 * i < npwx) emit(lane + 64 * i, xr[i]);
  } else {
    for (int g = lane; g < npwx; g += 64) emit(g, g < npw ? x[g] : cplx<T>{T(0), T(0)});
  }
}

// The projector rows of one k in LDS, read by all its bands: one workgroup per
// (k, group of up to kSBandsPerBlock rows).  Each row is handled by a half
// wavefront (32 lanes, two rows per wave at a time), which halves the cost of
// the lane reductions and of forming delta per row compared with a whole wave
// per row; each lane keeps its NPL plane waves (g = l + 32 i) of the row in
// registers.  Used when beta_k fits the LDS budget; it replaces the per-row
// L2 reads of beta (nproj rows per band, twice) by LDS reads.
constexpr int kSBandsPerBlock = 8;

// sum over the 32 lanes of each half of the wavefront, on every lane
template <class T>
__device__ __forceinline__ T half_sum(T v) {
  v += dpp<0xB1>(v);   // quad_perm 1,0,3,2
  v += dpp<0x4E>(v);   // quad_perm 2,3,0,1
  v += dpp<0x141>(v);  // row_half_mirror
  v += dpp<0x140>(v);  // row_mirror
  v += __shfl_xor(v, 16, 64);
  return v;
}

template <class T, int NP, int NPL>
__global__ __launch_bounds__(kSThreads) void spsi_lds_kernel(const cplx<T>* psi, cplx<T>* out, long kstride,
                                                             int nvec, const int* __restrict__ off,
                                                             const int* __restrict__ cnt,
                                                             const int* __restrict__ live,
                                                             const int* __restrict__ npw_k, int npwx, int nproj,
                                                             const cplx<T>* __restrict__ beta,
                                                             const cplx<T>* __restrict__ q,
                                                             const double* __restrict__ scale, double mult,
                                                             int per_xcd, int ngroup, int groups_per_k) {
  extern __shared__ char smem[];
  auto* qs = reinterpret_cast<cplx<T>*>(smem);        // q, nproj x nproj
  cplx<T>* bs = qs + nproj * nproj;                   // beta_k, nproj x npw_k (row stride npwx)
  const int bid = blockIdx.x;
  const int grp = (bid & 7) * per_xcd + (bid >> 3);
  if (grp >= ngroup) return;                          // whole workgroup: no barrier skipped
  const int k = grp / groups_per_k;
  const int r0 = (grp - k * groups_per_k) * kSBandsPerBlock;
  const int nrow = min(kSBandsPerBlock, (cnt ? cnt[k] : nvec) - r0);
  if (nrow <= 0) return;
  const int npw = npw_k[k];
  const cplx<T>* bk = beta + (long)k * nproj * npwx;
  for (int e = threadIdx.x; e < nproj * nproj; e += kSThreads) qs[e] = q[e];
  for (int p = 0; p < nproj; ++p)
    for (int g = threadIdx.x; g < npw; g += kSThreads) bs[p * npwx + g] = bk[(long)p * npwx + g];
  __syncthreads();
  const int l = threadIdx.x & 31, half = threadIdx.x >> 5;
  // both halves of a wave run the same number of iterations (the row index
  // is clamped and the surplus half masked), so the lane sums see every lane
  constexpr int NH = kSThreads / 32;
  for (int rb = 0; rb < nrow; rb += NH) {
    const int rr = rb + half;
    const bool on = rr < nrow;
    const int r = r0 + (on ? rr : 0);
    const int task = k * nvec + r;
    const bool act = on && !(live && !live[task]);
    const long row = (long)k * kstride + (long)((off ? off[k] : 0) + r) * npwx;
    const cplx<T>* x = psi + row;
    cplx<T>* y = out + row;
    cplx<T> xr[NPL];
#pragma unroll
    for (int i = 0; i < NPL; ++i) {
      const int g = l + 32 * i;
      xr[i] = (act && g < npw) ? x[g] : cplx<T>{T(0), T(0)};
    }
    T lr[NP], li[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) lr[p] = li[p] = T(0);
#pragma unroll
    for (int i = 0; i < NPL; ++i) {
      const int g = l + 32 * i;
      if (g < npw) {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
          if (p < nproj) {
            const cplx<T> bv = bs[p * npwx + g];
            lr[p] += bv.x * xr[i].x + bv.y * xr[i].y;
            li[p] += bv.x * xr[i].y - bv.y * xr[i].x;
          }
        }
      }
    }
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      if (p < nproj) {
        lr[p] = half_sum(lr[p]);
        li[p] = half_sum(li[p]);
      }
    }
    T dr[NP], di[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      dr[p] = di[p] = T(0);
      if (p < nproj) {
#pragma unroll
        for (int s2 = 0; s2 < NP; ++s2) {
          if (s2 < nproj) {
            const cplx<T> qq = qs[p * nproj + s2];
            dr[p] += qq.x * lr[s2] - qq.y * li[s2];
            di[p] += qq.x * li[s2] + qq.y * lr[s2];
          }
        }
      }
    }
    if (!act) continue;
    const T f = scale ? T(mult * scale[task]) : T(1);
#pragma unroll
    for (int i = 0; i < NPL; ++i) {
      const int g = l + 32 * i;
      if (g >= npwx) continue;
      if (g >= npw) {
        if (!scale) y[g] = {T(0), T(0)};
        continue;
      }
      cplx<T> v = xr[i];
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        if (p < nproj) {
          const cplx<T> bv = bs[p * npwx + g];
          v.x += dr[p] * bv.x - di[p] * bv.y;
          v.y += dr[p] * bv.y + di[p] * bv.x;
        }
      }
      if (scale) {
        const cplx<T> o = y[g];
        y[g] = {o.x + f * v.x, o.y + f * v.y};
      } else {
        y[g] = v;
      }
    }
  }
}

template <class T, int TW, bool P16>
void launch_spsi_mfma(pw_ctx* c, const VecSel& sel, const void* psi, void* out, const double* scale, double mult,
                      int nproj, const void* beta, const void* q, hipStream_t st) {
  const int groups_per_k = (sel.nvec + kSBands - 1) / kSBands;
  const int ngroup = groups_per_k * c->nk;
  const int per_xcd = (ngroup + 7) / 8;
  hipLaunchKernelGGL((spsi_mfma_kernel<T, TW, P16>), dim3(8u * (unsigned)per_xcd), dim3(kSThreads), 0, st,
                     (const cplx<T>*)psi, (cplx<T>*)out, sel.kstride, sel.nvec, sel.off, sel.cnt, sel.live, c->d_npw,
                     c->npwx, nproj, (const cplx<T>*)beta, (const cplx<T>*)q, scale, mult, per_xcd, ngroup,
                     groups_per_k);
}

template <class T, bool P16>
void launch_spsi_tw(pw_ctx* c, const VecSel& sel, const void* psi, void* out, const double* scale, double mult,
                    int nproj, const void* beta, const void* q, hipStream_t st) {
#define MKPW_SPSI(TW) launch_spsi_mfma<T, TW, P16>(c, sel, psi, out, scale, mult, nproj, beta, q, st)
  switch ((c->npwx + 63) / 64) {
    case 0:
    case 1: MKPW_SPSI(1); break;
    case 2: MKPW_SPSI(2); break;
    case 3: MKPW_SPSI(3); break;
    case 4: MKPW_SPSI(4); break;
    case 5: MKPW_SPSI(5); break;
    case 6: MKPW_SPSI(6); break;
    case 7: MKPW_SPSI(7); break;
    case 8: MKPW_SPSI(8); break;
    case 9:
    case 10:
    case 11:
    case 12: MKPW_SPSI(12); break;
    default: MKPW_SPSI(16); break;
  }
#undef MKPW_SPSI
}

constexpr size_t kSLdsBudget = 64 * 1024;

template <class T, int NP, int NPL>
void launch_spsi_lanes_t(pw_ctx* c, const VecSel& sel, const void* psi, void* out, const double* scale, double mult,
                   int nproj, const void* beta, const void* q, hipStream_t st) {
  if constexpr (NPL > 0) {
    const size_t lds_b = sizeof(cplx<T>) * ((size_t)nproj * nproj + (size_t)nproj * c->npwx);
    if (nproj > 0 && lds_b <= kSLdsBudget) {
      const int groups_per_k = (sel.nvec + kSBandsPerBlock - 1) / kSBandsPerBlock;
      const int ngroup = groups_per_k * c->nk;
      const int per_xcd = (ngroup + 7) / 8;
      hipLaunchKernelGGL((spsi_lds_kernel<T, NP, 2 * NPL>), dim3(8u * (unsigned)per_xcd), dim3(kSThreads), lds_b,
                         st, (const cplx<T>*)psi, (cplx<T>*)out, sel.kstride, sel.nvec, sel.off, sel.cnt, sel.live,
                         c->d_npw, c->npwx, nproj, (const cplx<T>*)beta, (const cplx<T>*)q, scale, mult, per_xcd,
                         ngroup, groups_per_k);
      return;
    }
  }
  const int ntask = sel.nvec * c->nk;
  const int nblk = (ntask + kSThreads / 64 - 1) / (kSThreads / 64);
  const int per_xcd = (nblk + 7) / 8;
  const size_t lds = sizeof(cplx<T>) * (size_t)std::max(1, nproj * nproj);
  hipLaunchKernelGGL((spsi_kernel<T, NP, NPL>), dim3(8u * (unsigned)per_xcd), dim3(kSThreads), lds, st,
                     (const cplx<T>*)psi, (cplx<T>*)out, sel.kstride, sel.nvec, sel.off, sel.cnt, sel.live, c->d_npw,
                     c->npwx, nproj, (const cplx<T>*)beta, (const cplx<T>*)q, scale, mult, per_xcd, ntask);
}

template <class T, int NP>
void launch_spsi_lanes(pw_ctx* c, const VecSel& sel, const void* psi, void* out, const double* scale, double mult,
                     int nproj, const void* beta, const void* q, hipStream_t st) {
  const int chunks = (c->npwx + 63) / 64;
  if (chunks <= 2)
    launch_spsi_lanes_t<T, NP, 2>(c, sel, psi, out, scale, mult, nproj, beta, q, st);
  else if (chunks <= 4)
    launch_spsi_lanes_t<T, NP, 4>(c, sel, psi, out, scale, mult, nproj, beta, q, st);
  else if (chunks <= 6)
    launch_spsi_lanes_t<T, NP, 6>(c, sel, psi, out, scale, mult, nproj, beta, q, st);
  else if (chunks <= 8)
    launch_spsi_lanes_t<T, NP, 8>(c, sel, psi, out, scale, mult, nproj, beta, q, st);
  else if (chunks <= 12)
    launch_spsi_lanes_t<T, NP, 12>(c, sel, psi, out, scale, mult, nproj, beta, q, st);
  else if (chunks <= 16)
    launch_spsi_lanes_t<T, NP, 16>(c, sel, psi, out, scale, mult, nproj, beta, q, st);
  else
    launch_spsi_lanes_t<T, NP, 0>(c, sel, psi, out, scale, mult, nproj, beta, q, st);
}

// Whether the matrix-core kernel takes less time than the others, which it does where
// the projectors are enough to fill its products: its time does not depend on them up
// to 8, theirs grows with them; it takes rows in groups of eight and holds them in
// tiles of 64 x {1 .. 8, 12, 16} plane waves.  By size (us, vector units / it):
//   * over 8 projectors: 1500 k x 8 rows [320], 9 projectors, FP64 359 / 71; not for
//     single complex64 rows that are long: 1500 k x 1 [832] 9 projectors 90 / 118;
//   * launches of up to 256 groups, where the latency of a group counts, from 4: 60 k x
//     20 [320] FP64 4 projectors 15 / 12, 8 22 / 12;
//   * FP64: [64 .. 256] from 5 (1500 k x 20 [256] 5 79 / 74, 4 70 / 67 but 4 63 / 69 at
//     128), [320] from 3 (4 122 / 93), [448] from 5 (4 151 / 152), [576, 640] from 8 (6
//     282 / 305), longer rows, whose projectors pass the LDS budget of the others, from 3;
//   * complex64: its products are no faster than half waves: 1500 k x 20 [320], 8
//     projectors 78 / 80, 4 48 / 67; rows of over 832 from 7.
// Groups of fewer than four rows fill their tiles in vain where rows are long: 1500 k x
// 1 [832], FP64, 8 projectors 82 / 109.
inline bool spsi_on_matrix_cores(int real, int nk, int nvec, int npwx, int nproj) {
  if (nproj > kSMfmaProj || npwx > kSMfmaRow) return false;
  if (nproj > 8) return real == 8 || nvec > 1 || npwx <= 512 || nproj > 12 || nk <= 512;
  if ((long)nk * ((nvec + kSBands - 1) / kSBands) <= 256) return nproj >= 4;
  if (npwx > 512 && nvec < 4) return false;
  if (real != 8) return npwx > 832 && nproj >= 7;
  return nproj >= (npwx <= 256 ? 5 : npwx <= 320 ? 3 : npwx <= 512 ? 5 : npwx <= 640 ? 8 : 3);
}

template <class T>
void launch_spsi_t(pw_ctx* c, const VecSel& sel, const void* psi, void* out, const double* scale, double mult,
                   int nproj, const void* beta, const void* q, hipStream_t st) {
  if (spsi_on_matrix_cores(sizeof(T), c->nk, sel.nvec, c->npwx, nproj)) {
    if (nproj <= 8)
      launch_spsi_tw<T, false>(c, sel, psi, out, scale, mult, nproj, beta, q, st);
    else
      launch_spsi_tw<T, true>(c, sel, psi, out, scale, mult, nproj, beta, q, st);
  } else if (nproj <= 8) {  // rows held in registers
    launch_spsi_lanes<T, 8>(c, sel, psi, out, scale, mult, nproj, beta, q, st);
  } else {  // one wave per row looping over the plane waves
    launch_spsi_lanes_t<T, kSMaxProj, 0>(c, sel, psi, out, scale, mult, nproj, beta, q, st);
  }
}

}  // namespace

pw_status launch_spsi(pw_ctx* c, pw_prec prec, const VecSel& sel, const void* psi, void* out, const double* scale,
                      double mult, hipStream_t st) {
  if (sel.nvec <= 0) return PW_OK;
  const int nproj = c->have_q ? c->nproj : 0;
  if (nproj > kSMaxProj) return set_err(c, PW_EINVAL, "overlap: more than 32 projectors");
  if (prec == PW_FP64)
    launch_spsi_t<double>(c, sel, psi, out, scale, mult, nproj, c->d_beta64, c->d_q64, st);
  else
    launch_spsi_t<float>(c, sel, psi, out, scale, mult, nproj, c->d_beta32, c->d_q32, st);
  return check_launch(c, "s_psi", st);
}

}  // namespace mkpw

extern "C" pw_status pw_s_psi(pw_ctx* c, pw_prec prec, int nbnd, const void* psi, void* spsi) {
  using namespace mkpw;
  if (!c) return PW_EINVAL;
  if (c->host_only) return set_err(c, PW_ESTATE, "host-only context runs no device work");
  if (!c->have_k) return set_err(c, PW_ESTATE, "set k-points before s_psi");
  if (prec != PW_FP64 && prec != PW_MIXED) return set_err(c, PW_EINVAL, "unknown precision");
  if (nbnd <= 0 || nbnd > 65535) return set_err(c, PW_EINVAL, "nbnd must be in [1, 65535]");
  if (!psi || !spsi) return set_err(c, PW_EINVAL, "null psi or spsi");
  (void)hipSetDevice(c->device);
  VecSel sel;
  sel.nvec = nbnd;
  sel.kstride = (long)nbnd * c->npwx;
  return launch_spsi(c, prec, sel, psi, spsi, nullptr, 0.0, c->stream);
}
