// Batched H|psi> with the local potential as a dense matrix per k on the
// matrix cores.
//
// The local term of Sec. 3's H application, scatter -> inverse transform ->
// V(r) -> forward transform -> gather, is on the sphere of k exactly the sum
//   (V psi)(G') = sum_G V~[(m_G' - m_G) mod N] psi(G),
// V~ the forward transform of V(r) with 1/N_r (Eqs. zfft .. fwFFT regrouped):
// a complex npw x npw matrix times the k's vectors.  Only the differences |d| < W
// of the Miller window occur, so the matrix is never formed: its entries are read
// from a box of V~ values in LDS (one half of it, V being real: 74 KB in FP64 at a
// window of 11).  8 npw^2 flop per row are no more than the transforms' at npw of a
// few hundred (dense_faster says where the line lies), and they run on the matrix cores, where the transforms keep the
// vector units 40% (FP64) to 93% (complex64) busy.
//
// What bounds it: the matrix cores' issue.  Every vector instruction costs them 2
// to 6 cycles (measured beside v_mfma_f64_16x16x4, 64 cycles, and
// v_mfma_f32_16x16x4, 32), so an entry takes three (address, sign, negation) and
// serves up to 24 vectors, and psi is staged in the form the products read.  On
// MI355X, us (transforms on the context's mesh / on the smallest mesh / this):
//   512 k x 20 vectors, npw 305, FP64       379 /  316 /  163  matrix cores 66% busy
//   1728 k x 24 vectors, npw 469, FP64     4109 / 1860 / 1420  71%
//   2048 k x 16 vectors, npw 305, complex64 870 /  461 /  258  69%
//   1728 k x 24 vectors, npw 469, complex64 1820 / 902 /  714  70%
// (busy: of the cycles of the whole launch, its start and end among them; the rest:
// uneven row tiles, vector instructions, the start, the projectors and the output of a
// workgroup).  psi is read twice, for the product and for the kinetic term: 1.05 GB of
// HBM traffic at 1728 k in FP64, 0.74 TB/s.  Rounding is below the
// transforms' (complex64 3.6e-8 of the result against 5.6e-8 to 8.4e-8).  Tried
// and dropped: entries gathered from L2 (1640 us at 1728 k, FP64: the vector
// memory path takes 57 to 90 cycles a gather), rows in Miller order with the
// results put back in order in LDS (166 against 162 us: the gathers' bank
// conflicts are not what bounds it), 16 waves a workgroup (1514), persistent
// workgroups that keep the box (1480).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <string>
#include <type_traits>

#include "hpsi_dense_shape.hpp"
#include "internal.hpp"

namespace mkpw {

namespace {

// D (16 x 16) += A (16 x 4) B (4 x 16), one wave: lane l holds A[l % 16][l / 16]
// and B[l / 16][l % 16]; item r of the result is row Mf::row(r, l / 16), column
// l % 16.  In FP64 also D (16 x 4) += A (16 x 4) B (4 x 4), a quarter of the
// columns in a quarter of the time (16 of 64 cycles; both reach 69 TFLOP/s),
// from the same A: it is four blocks of 4 x 4, lane l holds B[l / 16][l % 4]
// whatever its block, and the result is row 4 ((l / 4) % 4) + l / 16, column
// l % 4.
template <class T>
struct Mf;
template <>
struct Mf<double> {
  typedef double acc __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ acc mul(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int r, int kq) { return 4 * r + kq; }
  static __device__ __forceinline__ double mul4(double a, double b, double c) {
    return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
  }
};
template <>
struct Mf<float> {
  typedef float acc __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ acc mul(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int r, int kq) { return 4 * kq + r; }
  static __device__ __forceinline__ float mul4(float, float, float c) { return c; }  // not used
};

constexpr int kGS = kDenseGS, kTS = kDenseTS;

// y, negated where s is negative
__device__ __forceinline__ float flip(float y, int s) { return __int_as_float(__float_as_int(y) ^ (s & 0x80000000)); }
__device__ __forceinline__ double flip(double y, int s) {
  return __hiloint2double(__double2hiint(y) ^ (s & 0x80000000), __double2loint(y));
}

// |a - b| of two offsets >= 0 in one instruction
__device__ __forceinline__ unsigned abs_diff(int a, int b) {
  unsigned d;
  asm("v_sad_u32 %0, %1, %2, 0" : "=v"(d) : "v"(a), "v"(b));
  return d;
}

// complex value at an LDS byte address that is a multiple of its size (one read
// of that width)
template <class T>
__device__ __forceinline__ cplx<T> lds_read(unsigned addr) {
  typedef T pair __attribute__((ext_vector_type(2)));
  const pair v = *(const __attribute__((address_space(3))) pair*)(size_t)addr;
  return {v.x, v.y};
}

template <int N>
using ic = std::integral_constant<int, N>;

constexpr int kMaxProjDense = 16;

template <class T>
struct DenseArgs {
  const int* npw;
  const int* mkey;  // packed Miller indices, library order
  const double* kin;
  int npwx;
  VecSel sel;
  int nproj;
  const cplx<T>* beta;
  const cplx<T>* dij;
  // projectors nproj .. nproj + nextra - 1: rows of a term alpha_k |row> <row|
  int nextra;
  const cplx<T>* extra;
  const double* alpha;
  const cplx<T>* box;  // V~ of the Miller differences of linear offset 0 .. nhalf - 1
  int s2, s3, nhalf;   // strides of the box
  const cplx<T>* psi;
  cplx<T>* hpsi;
  int nbt, nsplit;  // band blocks and row splits per k
  int per_xcd, ntask;
};

// Linear offset of a Miller triple (shifted by 512 per axis, so not negative;
// below 2^26 for boxes that fit in LDS); the offset of a difference is the
// difference of the offsets, and of -d the negative
__device__ __forceinline__ int box_lin(int key, int s2, int s3) {
  return (((key >> 20) & 1023) * s2 + ((key >> 10) & 1023)) * s3 + (key & 1023);
}

// One workgroup of NW waves: one k, up to 8 NGM of its selected vectors, up to
// 16 NW RTM rows G'.
template <class T, int NW, int NGM, int RTM>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2))) void hpsi_dense_kernel(
    DenseArgs<T> a) {
  using M = Mf<T>;
  typedef typename M::acc acc_t;
  constexpr int NB = 8 * NGM, KC = dense_kc(NW, NGM, RTM), BS = dense_bs(NW, NGM, RTM, sizeof(T)), NT = NW * 64;
  constexpr int CS = (int)sizeof(cplx<T>);
  constexpr int kSteps = KC / 4;
  constexpr int kFetch = (NB * KC + NT - 1) / NT;  // staged values per work-item
  // chunks that psi is loaded ahead of its use: a chunk of one group is short
  // against a load
  constexpr int kAhead = NGM == 1 && RTM > 2 ? 2 : 1;
  constexpr int kL = (kSteps + NW - 1) / NW;  // steps of a chunk that a wave sums for the projectors
  extern __shared__ __align__(16) char smem[];
  const int npwx = a.npwx, nproj = a.nproj, nall = nproj + a.nextra;
  const DenseLds L = dense_lds(sizeof(T), NW, NGM, RTM, npwx, a.nhalf, nproj, nall);
  T* buf = reinterpret_cast<T*>(smem + L.buf);  // [2][NB][BS]
  int* wcol = reinterpret_cast<int*>(smem + L.wcol);  // byte offset of each column G, past npw that of G = 0
  int* slot = reinterpret_cast<int*>(smem + L.slot);  // [NB] the selected vectors, then their number

  // consecutive tasks run on one XCD, so the blocks of a k share its L2
  const int task = (blockIdx.x & 7) * a.per_xcd + (blockIdx.x >> 3);
  if (task >= a.ntask) return;
  const int per_k = a.nbt * a.nsplit;
  const int ik = task / per_k, sub = task - ik * per_k;
  const int bt = sub / a.nsplit, split = sub - bt * a.nsplit;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, kq = lane >> 4, part = l16 >> 3, part4 = (lane >> 1) & 1;
  // the vectors of this block: the selected ones of the k with ranks
  // [bt NB, bt NB + NB)
  const int cnt = a.sel.cnt ? a.sel.cnt[ik] : a.sel.nvec;
  int nact = cnt - bt * NB;
  if (nact <= 0) return;
  const bool listed = a.sel.live != nullptr;
  if (listed) {
    const int* lv = a.sel.live + (long)ik * a.sel.nvec;
    if (wave == 0) {
      int base = 0;
      for (int i0 = 0; i0 < cnt; i0 += 64) {
        const bool on = i0 + lane < cnt && lv[i0 + lane] != 0;
        const unsigned long long m = __ballot(on);
        const int r = base + __popcll(m & ((1ull << lane) - 1ull)) - bt * NB;
        if (on && r >= 0 && r < NB) slot[r] = i0 + lane;
        base += __popcll(m);
      }
      if (lane == 0) slot[NB] = base;
    }
    __syncthreads();
    nact = __builtin_amdgcn_readfirstlane(slot[NB]) - bt * NB;
    if (nact <= 0) return;
  }
  nact = min(nact, NB);
  // groups of 8 vectors: the first nfull as 16 columns each (the real parts of
  // the 8, then their imaginary parts), in FP64 the rest as ntail sets of 4 (the
  // real parts of two vectors, then their imaginary parts)
  constexpr bool kTail = sizeof(T) == 8;
  const int nset = kTail ? (nact + 1) >> 1 : ((nact + 7) >> 3) * 4;
  const int nfull = nset >> 2, ntail = nset & 3;
  const int npw = a.npw[ik];
  const int* key = a.mkey + (long)ik * npwx;
  // vector b of the block
  const long kbase = (long)ik * a.sel.kstride + (long)(a.sel.off ? a.sel.off[ik] : 0) * npwx;
  auto vec = [&](int b) { return kbase + (long)(listed ? slot[b] : bt * NB + b) * npwx; };

  // staging of psi: value tid + q NT of a chunk
  const cplx<T>* src[kFetch];
  bool son[kFetch];
  cplx<T> pre[kAhead][kFetch];
#pragma unroll
  for (int q = 0; q < kFetch; ++q) {
    const int b = (tid + q * NT) / KC;
    son[q] = b < nact;
    src[q] = a.psi + vec(son[q] ? b : 0);
  }
  auto fetch = [&](int c, cplx<T>(&x)[kFetch]) {
    const int g = dense_psi_index(c, KC, tid & (KC - 1), npw);
#pragma unroll
    for (int q = 0; q < kFetch; ++q) x[q] = src[q][g];
  };
  auto store = [&](int c, const cplx<T>(&x)[kFetch]) {
    const bool in = c * KC + (tid & (KC - 1)) < npw;
#pragma unroll
    for (int q = 0; q < kFetch; ++q) {
      const int e = tid + q * NT;
      const bool ok = in && son[q];
      if (NB * KC % NT == 0 || e < NB * KC) {
        T* d = buf + (c & 1) * NB * BS + e / KC * BS + 3 * (e % KC);
        d[0] = ok ? -x[q].y : T(0);
        d[1] = ok ? x[q].x : T(0);
        d[2] = ok ? x[q].y : T(0);
      }
    }
  };
  const int nch = (npw + KC - 1) / KC;
  if (nch > 0) fetch(0, pre[0]);
  if constexpr (kAhead == 2) {
    if (nch > 1) fetch(1, pre[1]);
  }
  // rows G' of this lane
  const int ntile = (npw + 15) >> 4;
  const int t0 = split * NW + wave, tstep = a.nsplit * NW;
  int prow[RTM];
#pragma unroll
  for (int i = 0; i < RTM; ++i) {
    const int g = (t0 + i * tstep) * 16 + l16;
    prow[i] = key[g < npw ? g : 0];
  }
  const bool last = t0 + (RTM - 1) * tstep < ntile;
  {
    cplx<T>* boxs = reinterpret_cast<cplx<T>*>(smem);
    for (int e0 = tid; e0 < a.nhalf; e0 += 8 * NT) {  // eight loads in flight
      cplx<T> t[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) t[u] = a.box[min(e0 + u * NT, a.nhalf - 1)];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (e0 + u * NT < a.nhalf) boxs[e0 + u * NT] = t[u];
    }
    cplx<T>* dl = reinterpret_cast<cplx<T>*>(smem + L.dl);
    for (int e = tid; e < nproj * nproj; e += NT) dl[e] = a.dij[e];
    for (int j = tid; j < dense_ncol(KC, npwx); j += NT) wcol[j] = box_lin(key[j < npw ? j : 0], a.s2, a.s3) * CS;
  }
#pragma unroll
  for (int i = 0; i < RTM; ++i) prow[i] = box_lin(prow[i], a.s2, a.s3) * CS;
  if (nch > 0) store(0, pre[0]);
  __syncthreads();

  acc_t acc[NGM][RTM], lam[NGM];
#pragma unroll
  for (int g = 0; g < NGM; ++g) {
    lam[g] = acc_t{0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < RTM; ++i) acc[g][i] = acc_t{0, 0, 0, 0};
  }
  // row p of the k's projectors, both kinds
  auto proj_row = [&](int p) {
    return p < nproj ? a.beta + ((long)ik * nproj + p) * npwx : a.extra + ((long)ik * a.nextra + p - nproj) * npwx;
  };
  const cplx<T>* brow = nall > 0 ? proj_row(l16 < nall ? l16 : 0) : nullptr;
  // the sum over G for NF full groups and NQ sets of the next one (the same for
  // the whole workgroup, so that the steps of a chunk are straight-line code);
  // set t of group NF is summed in component t of that group's accumulators
  auto sum_g = [&](auto nf, auto nq) {
    constexpr int NF = decltype(nf)::value, NQ = decltype(nq)::value, NG = NF + NQ;
    constexpr int G4 = NF < NGM ? NF : 0;  // the group of the sets
    constexpr int AH = dense_steps_ahead(NG, RTM);
    cplx<T> v[AH][RTM];
    int sg[AH][RTM];
    // V is real, so V~(-d) is the conjugate of V~(d): the box holds one half,
    // and the sign of the offset goes to the imaginary part.  (The box is at
    // LDS address 0: the kernel has no static LDS.)
    auto gather = [&](int h, int i, int w) {
      sg[h][i] = prow[i] - w;
      v[h][i] = lds_read<T>(abs_diff(prow[i], w));
    };
#pragma unroll
    for (int h = 0; h < AH; ++h) {
      const int w = wcol[4 * h + kq];
#pragma unroll
      for (int i = 0; i < RTM; ++i) gather(h, i, w);
    }
    int w = wcol[4 * AH + kq];  // of the next entry to read
    // projector overlaps lambda = beta^H psi (Eq. lambdah), rows = projectors:
    // the steps are dealt to the waves
    auto mine = [&](int c) { return nall > 0 && (kSteps >= NW || (c & (NW / kSteps - 1)) == wave / kSteps); };
    auto first_step = [&]() { return kSteps >= NW ? wave : wave & (kSteps - 1); };
    auto load_beta = [&](int c, cplx<T>(&x)[kL]) {
      if (nall > 0 && c < nch) {
#pragma unroll
        for (int u = 0; u < kL; ++u) {
          const int j = c * KC + 4 * (first_step() + NW * u) + kq;
          x[u] = brow[j < npw ? j : 0];
        }
      }
    };
    cplx<T> bet[kAhead][kL];
    if constexpr (kAhead == 2) {
      load_beta(0, bet[0]);
      load_beta(1, bet[1]);
    }
    // one chunk; `slot` (c modulo kAhead) names the registers its successor's
    // values arrive in
    auto chunk = [&](int c, auto slotc) {
      constexpr int SL = decltype(slotc)::value;
      cplx<T>(&bl)[kL] = bet[SL];
      const T* bs = buf + (c & 1) * NB * BS + 3 * kq;
      const T* bs16 = bs + (l16 & 7) * BS + part;
      const T* bs4 = bs + (NF * 8 + (lane & 1)) * BS + part4;
      // a lane's columns of step st: Re L meets (re, im), Im L meets (-im, re)
      struct Col {
        T b2, b1;
      };
      auto load_b = [&](Col(&x)[NG], int st) {
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          const T* q = (g < NF ? bs16 + g * 8 * BS : bs4 + 2 * (g - NF) * BS) + 12 * st;
          x[g] = {q[0], q[1]};
        }
      };
      Col b[AH][NG];
#pragma unroll
      for (int h = 0; h < AH; ++h) load_b(b[h], h);
      if (c + kAhead < nch) fetch(c + kAhead, pre[SL]);
      if constexpr (kAhead == 1) load_beta(c, bl);
      constexpr int kU = kSteps < 8 ? kSteps : 8, kH = AH;  // steps unrolled
      for (int s0 = 0; s0 < kSteps; s0 += kU) {
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          const int s = s0 + u, h = u % kH;
          Col x[NG];
#pragma unroll
          for (int g = 0; g < NG; ++g) x[g] = b[h][g];
          if (kSteps > kU || u + kH < kSteps) load_b(b[h], s + kH);
          const int wn = wcol[c * KC + 4 * (s + kH + 1) + kq];
          // a tile's next entry is read as soon as this step's products have
          // used this one
          auto tile = [&](int i) {
            const T y = flip(v[h][i].y, sg[h][i]);
#pragma unroll
            for (int g = 0; g < NF; ++g) acc[g][i] = M::mul(v[h][i].x, x[g].b1, acc[g][i]);
#pragma unroll
            for (int t = 0; t < NQ; ++t) acc[G4][i][t] = M::mul4(v[h][i].x, x[NF + t].b1, acc[G4][i][t]);
#pragma unroll
            for (int g = 0; g < NF; ++g) acc[g][i] = M::mul(y, x[g].b2, acc[g][i]);
#pragma unroll
            for (int t = 0; t < NQ; ++t) acc[G4][i][t] = M::mul4(y, x[NF + t].b2, acc[G4][i][t]);
          };
#pragma unroll
          for (int i = 0; i < RTM - 1; ++i) {
            tile(i);
            gather(h, i, w);
          }
          // (read by every wave: a read under the branch would make the next
          // step wait for it)
          if (last) tile(RTM - 1);
          gather(h, RTM - 1, w);
          w = wn;
        }
      }
      if (mine(c)) {
        const int ls0 = first_step();
#pragma unroll
        for (int u = 0; u < kL; ++u) {
          const T lx = l16 < nall ? bl[u].x : T(0), ly = l16 < nall ? -bl[u].y : T(0);
          Col x[NG];
          load_b(x, ls0 + NW * u);
#pragma unroll
          for (int g = 0; g < NF; ++g) {
            lam[g] = M::mul(lx, x[g].b1, lam[g]);
            lam[g] = M::mul(ly, x[g].b2, lam[g]);
          }
#pragma unroll
          for (int t = 0; t < NQ; ++t) {
            lam[G4][t] = M::mul4(lx, x[NF + t].b1, lam[G4][t]);
            lam[G4][t] = M::mul4(ly, x[NF + t].b2, lam[G4][t]);
          }
        }
      }
      if constexpr (kAhead == 2) load_beta(c + 2, bl);
      if (c + 1 < nch) store(c + 1, pre[(SL + 1) % kAhead]);
      __syncthreads();
    };
    for (int c = 0; c < nch; c += kAhead) {
      chunk(c, ic<0>{});
      if constexpr (kAhead == 2) {
        if (c + 1 < nch) chunk(c + 1, ic<1>{});
      }
    }
  };
  auto sum_nf = [&](auto nf) {
    constexpr int NF = decltype(nf)::value;
    if constexpr (NF > 0) {
      if (ntail == 0) sum_g(nf, ic<0>{});
    }
    if constexpr (kTail && NF < NGM) {
      if (ntail == 1) sum_g(nf, ic<1>{});
      if (ntail == 2) sum_g(nf, ic<2>{});
      if (ntail == 3) sum_g(nf, ic<3>{});
    }
  };
  if (nfull == 0) sum_nf(ic<0>{});
  if (nfull == 1) sum_nf(ic<1>{});
  if constexpr (NGM >= 2) {
    if (nfull == 2) sum_nf(ic<2>{});
  }
  if constexpr (NGM >= 3) {
    if (nfull == 3) sum_nf(ic<3>{});
  }
  // f(r, row, vector of the group, part) for the items of this lane's
  // accumulators of group g
  const int row4 = (lane & 12) + kq;
  auto items = [&](int g, auto f) {
    if (g < nfull) {
#pragma unroll
      for (int r = 0; r < 4; ++r) f(r, M::row(r, kq), l16 & 7, part);
    } else if (kTail && g == nfull) {
#pragma unroll
      for (int t = 0; t < 3; ++t)
        if (t < ntail) f(t, row4, 2 * t + (lane & 1), part4);
    }
  };

  // gamma = D lambda (Eq. gamma), then sum_p beta_p gamma_p (Eq. finalnl) as
  // more columns of the same product
  if (nall > 0) {
    cplx<T> x[RTM];
    auto beta_rows = [&](int p0) {
      const cplx<T>* pr = proj_row(p0 + kq < nall ? p0 + kq : 0);
#pragma unroll
      for (int i = 0; i < RTM; ++i) {
        const int g = (t0 + i * tstep) * 16 + l16;
        x[i] = pr[g < npw ? g : 0];
      }
    };
    beta_rows(0);
    cplx<T>* red = reinterpret_cast<cplx<T>*>(smem);                // [NW][16][NB]
    cplx<T>* ls = reinterpret_cast<cplx<T>*>(smem) + NW * 16 * NB;  // lambda [16][NB]
    cplx<T>* gs = ls + 16 * NB;                                     // gamma [NB][kGS]
    const cplx<T>* dl = reinterpret_cast<const cplx<T>*>(smem + L.dl);
#pragma unroll
    for (int g = 0; g < NGM; ++g)
      items(g, [&](int r, int p, int b, int pt) {
        reinterpret_cast<T*>(red + (wave * 16 + p) * NB + g * 8 + b)[pt] = lam[g][r];
      });
    __syncthreads();
    for (int e = tid; e < 16 * NB; e += NT) {
      const int p = e / NB, b = e - p * NB;
      cplx<T> y = {T(0), T(0)};
#pragma unroll
      for (int w = 0; w < NW; ++w) y = cadd(y, red[(w * 16 + p) * NB + b]);
      ls[e] = y;
    }
    __syncthreads();
    for (int e = tid; e < 16 * NB; e += NT) {
      const int b = e >> 4, p = e & 15;
      cplx<T> y = {T(0), T(0)};
      if (p < nproj) {
        for (int q = 0; q < nproj; ++q) y = cfma(dl[p * nproj + q], ls[q * NB + b], y);
      } else if (p < nall) {
        const T al = (T)a.alpha[ik];
        y = {al * ls[p * NB + b].x, al * ls[p * NB + b].y};
      }
      gs[b * kGS + p] = y;
    }
    __syncthreads();
    for (int p0 = 0; p0 < nall; p0 += 4) {
      const int p = p0 + kq;
      cplx<T> y[RTM];
#pragma unroll
      for (int i = 0; i < RTM; ++i) {
        const bool ok = (t0 + i * tstep) * 16 + l16 < npw && p < nall;
        y[i] = {ok ? x[i].x : T(0), ok ? x[i].y : T(0)};
      }
      if (p0 + 4 < nall) beta_rows(p0 + 4);
#pragma unroll
      for (int g = 0; g < NGM; ++g) {
        if (g < nfull) {
          const cplx<T> b = gs[(g * 8 + (l16 & 7)) * kGS + p];
          const T b1 = part ? b.y : b.x, b2 = part ? b.x : -b.y;
#pragma unroll
          for (int i = 0; i < RTM; ++i) acc[g][i] = M::mul(y[i].x, b1, acc[g][i]);
#pragma unroll
          for (int i = 0; i < RTM; ++i) acc[g][i] = M::mul(y[i].y, b2, acc[g][i]);
        } else if (kTail && g == nfull) {
#pragma unroll
          for (int t = 0; t < 3; ++t) {
            if (t < ntail) {
              const cplx<T> b = gs[(g * 8 + 2 * t + (lane & 1)) * kGS + p];
              const T b1 = part4 ? b.y : b.x, b2 = part4 ? b.x : -b.y;
#pragma unroll
              for (int i = 0; i < RTM; ++i) acc[g][i][t] = M::mul4(y[i].x, b1, acc[g][i][t]);
#pragma unroll
              for (int i = 0; i < RTM; ++i) acc[g][i][t] = M::mul4(y[i].y, b2, acc[g][i][t]);
            }
          }
        }
      }
    }
    __syncthreads();  // gamma has been read
  }

  // add the kinetic term and write: each 16 x 8 tile goes through this wave's
  // part of LDS, so that 16 lanes read and write 16
  // consecutive plane waves of a vector; psi of the next tile is loaded
  // before this one is written
  cplx<T>* tl = reinterpret_cast<cplx<T>*>(smem) + wave * NB * kTS;
  cplx<T> pn[NGM][2];
  T kn = T(0);
  long row[NGM][2];
#pragma unroll
  for (int g = 0; g < NGM; ++g)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int b = g * 8 + kq + 4 * u;
      row[g][u] = vec(b < nact ? b : 0) + l16;
    }
  auto load_psi = [&](int t) {
    kn = (T)a.kin[(long)ik * npwx + t * 16 + l16];
#pragma unroll
    for (int g = 0; g < NGM; ++g)
#pragma unroll
      for (int u = 0; u < 2; ++u) pn[g][u] = a.psi[row[g][u] + t * 16];
  };
  if (t0 < ntile) load_psi(t0);
#pragma unroll
  for (int i = 0; i < RTM; ++i) {
    const int t = t0 + i * tstep;
    if (t < ntile) {
      cplx<T> pc[NGM][2];
      const T kk = kn;
#pragma unroll
      for (int g = 0; g < NGM; ++g)
#pragma unroll
        for (int u = 0; u < 2; ++u) pc[g][u] = pn[g][u];
      if (i + 1 < RTM && t + tstep < ntile) load_psi(t + tstep);
      const bool ok = t * 16 + l16 < npw;
#pragma unroll
      for (int g = 0; g < NGM; ++g)
        items(g, [&](int r, int j, int b, int pt) {
          reinterpret_cast<T*>(tl + (g * 8 + b) * kTS + j)[pt] = acc[g][i][r];
        });
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int g = 0; g < NGM; ++g)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const cplx<T> h = tl[(g * 8 + kq + 4 * u) * kTS + l16];
          if (g * 8 + kq + 4 * u < nact)
            a.hpsi[row[g][u] + t * 16] = {ok ? h.x + kk * pc[g][u].x : T(0), ok ? h.y + kk * pc[g][u].y : T(0)};
        }
      __builtin_amdgcn_wave_barrier();
    }
  }
  // the padding past the last tile
  if (split == 0) {
    const int z0 = ntile * 16;
    for (int e = tid; e < nact * (npwx - z0); e += NT) {
      const int b = e / (npwx - z0);
      a.hpsi[vec(b) + z0 + (e - b * (npwx - z0))] = {T(0), T(0)};
    }
  }
}

template <class T, int NW, int NGM, int RTM>
pw_status launch_inst(pw_ctx* c, DenseArgs<T>& a, hipStream_t st) {
  const size_t lds = dense_lds(sizeof(T), NW, NGM, RTM, a.npwx, a.nhalf, a.nproj, a.nproj + a.nextra).bytes;
  const void* kern = (const void*)hpsi_dense_kernel<T, NW, NGM, RTM>;
  pw_status s = ensure_lds_limit(c, kern, lds);
  if (s != PW_OK) return s;
  hipLaunchKernelGGL((hpsi_dense_kernel<T, NW, NGM, RTM>), dim3(8u * (unsigned)a.per_xcd), dim3(NW * 64), lds, st, a);
  return check_launch(c, "h_psi", st);
}

template <class T, int NW, int NGM>
pw_status launch_rt(pw_ctx* c, DenseArgs<T>& a, int rt, hipStream_t st) {
  if constexpr (NW == 4) {
    if (rt == 5) return launch_inst<T, NW, NGM, 5>(c, a, st);
    if (rt == 6) return launch_inst<T, NW, NGM, 6>(c, a, st);
    if constexpr (sizeof(T) == 4) {
      if (rt == 7) return launch_inst<T, NW, NGM, 7>(c, a, st);
      if (rt == 8) return launch_inst<T, NW, NGM, 8>(c, a, st);
    }
  }
  switch (rt) {
    case 1: return launch_inst<T, NW, NGM, 1>(c, a, st);
    case 2: return launch_inst<T, NW, NGM, 2>(c, a, st);
    case 3: return launch_inst<T, NW, NGM, 3>(c, a, st);
    default: return launch_inst<T, NW, NGM, 4>(c, a, st);
  }
}

template <class T, int NW>
pw_status launch_ng(pw_ctx* c, DenseArgs<T>& a, int ngm, int rt, hipStream_t st) {
  return ngm == 1 ? launch_rt<T, NW, 1>(c, a, rt, st) : ngm == 2 ? launch_rt<T, NW, 2>(c, a, rt, st)
                                                                 : launch_rt<T, NW, 3>(c, a, rt, st);
}

template <class T>
pw_status launch_t(pw_ctx* c, const VecSel& sel, const void* psi, void* hpsi, hipStream_t st, const ProjTerm* extra) {
  const bool fp64 = sizeof(T) == 8;
  DenseArgs<T> a;
  a.npw = c->d_npw;
  a.mkey = c->d_mkey;
  a.kin = c->d_kin;
  a.npwx = c->npwx;
  a.sel = sel;
  a.nproj = c->have_proj ? c->nproj : 0;
  a.beta = (const cplx<T>*)(fp64 ? c->d_beta64 : c->d_beta32);
  a.dij = (const cplx<T>*)(fp64 ? c->d_dij64 : c->d_dij32);
  a.nextra = extra ? extra->n : 0;
  a.extra = extra ? (const cplx<T>*)extra->rows : nullptr;
  a.alpha = extra ? extra->alpha : nullptr;
  a.box = (const cplx<T>*)(fp64 ? c->d_box64 : c->d_box32);
  a.s2 = 2 * c->wy - 1;
  a.s3 = 2 * c->wz - 1;
  a.nhalf = hpsi_dense_box(c);
  a.psi = (const cplx<T>*)psi;
  a.hpsi = (cplx<T>*)hpsi;
  if ((long)c->nk * sel.nvec <= 0) return PW_OK;
  const auto [nw, ngm, rt, nbt, nsplit] =
      dense_shape(sizeof(T), c->nk, sel.nvec, c->npwmax, a.npwx, a.nhalf, a.nproj, a.nproj + a.nextra);
  a.nbt = nbt;
  a.nsplit = nsplit;
  const long ntask = (long)c->nk * nbt * nsplit;
  if (ntask > (1L << 30)) return set_err(c, PW_EINVAL, "too many (k, band) rows in one call");
  a.ntask = (int)ntask;
  a.per_xcd = (int)((ntask + 7) / 8);
  pw_status s = nw == 4 ? launch_ng<T, 4>(c, a, ngm, rt, st) : launch_ng<T, 8>(c, a, ngm, rt, st);
  if (s != PW_OK) return s;
  c->last_hpsi_variant = 6;
  c->last_hpsi_slab = 0;
  c->last_hpsi_threads = nw * 64;
  return PW_OK;
}

}  // namespace

// Entries of the box with a linear offset >= 0, or 0 where it does not fit in LDS
// with the rest
int hpsi_dense_box(const pw_ctx* c) {
  const long n = (long)(2 * c->wx - 1) * (2 * c->wy - 1) * (2 * c->wz - 1);
  const long half = (n + 1) / 2;
  if (half > (long)(kDenseLdsPerCu / sizeof(cplx<double>))) return 0;
  return dense_lds(8, 8, 1, 3, c->npwx, (int)half, kMaxProjDense, kMaxProjDense).bytes <= kDenseLdsPerCu ? (int)half : 0;
}

// Whether H|psi> of this call takes the dense product rather than the transforms
// on the smallest mesh
bool hpsi_takes_dense(const pw_ctx* c, pw_prec prec, const VecSel& sel, int nextra) {
  if (!c->d_box64 || !c->d_box32) return false;
  if (c->hpsi_variant != 0 || c->hpsi_slab != 0 || c->hpsi_threads != 0) return false;  // a transform shape is asked for
  const int nproj = c->have_proj ? c->nproj : 0;
  if (nproj + nextra > kMaxProjDense) return false;  // lambda is one tile of rows
  return dense_faster(prec == PW_FP64 ? 8 : 4, c->nk, sel.nvec, c->npwmax, c->npwx, hpsi_dense_box(c), nproj,
                      nproj + nextra, c->kmesh ? c->kmesh : c->fft[0], std::max(c->wx, std::max(c->wy, c->wz)));
}

pw_status launch_hpsi_dense(pw_ctx* c, pw_prec prec, const VecSel& sel, const void* psi, void* hpsi, hipStream_t st,
                            const ProjTerm* extra) {
  return prec == PW_FP64 ? launch_t<double>(c, sel, psi, hpsi, st, extra) : launch_t<float>(c, sel, psi, hpsi, st, extra);
}

}  // namespace mkpw
