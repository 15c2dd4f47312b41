// Launch shapes of the dense H|psi> product (hpsi_dense.hip) and the ranges of its
// LDS and of psi that a shape reads.  Plain arithmetic, so that a host program can
// walk every shape without a GPU.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstddef>

#ifndef __HIPCC__
#define MKPW_HD
#else
#define MKPW_HD __host__ __device__
#endif

namespace mkpw {

constexpr size_t kDenseLdsPerCu = 160 * 1024;
constexpr int kDenseCus = 256;
constexpr int kDenseGS = 20;  // stride of gamma's rows
constexpr int kDenseTS = 17;  // stride of the rows of a transposed output tile

// plane waves of psi staged in LDS at a time: few where two workgroups share a
// CU's LDS and a chunk has work enough to cover the next one's loads, more for
// the small row blocks of launches that leave the chip part empty
MKPW_HD constexpr int dense_kc(int nw, int ngm, int rt) {
  return rt <= 2 ? (ngm == 1 ? 128 : ngm == 2 ? 64 : 32) : nw == 4 && ngm == 3 ? 16 : 32;
}
// Reals of a staged row of psi.  A plane wave takes three, (-im, re, im), so that
// a lane reads its two columns (b2, b1 of the products) as two neighbours and
// selects nothing: vector instructions take the matrix cores' issue slots (one
// between two FP64 products costs 6 cycles of 65, eight cost 20).  The pad of 32
// bytes spreads the rows of a step over the banks.
MKPW_HD constexpr int dense_bs(int nw, int ngm, int rt, int real) { return 3 * dense_kc(nw, ngm, rt) + 32 / real; }

// A row of psi is npwx long, a multiple of 64, and a chunk may be 128: the last one
// of a row then reaches past it.  Staged value t of chunk c is element
// dense_psi_index of its row; past the sphere it is the first one, which is stored
// as zero.
MKPW_HD constexpr int dense_psi_index(int c, int kc, int t, int npw) { return c * kc + t < npw ? c * kc + t : 0; }

// steps an entry of the box is read ahead of its use: one where a step has
// products enough to cover the read, more for a small block (ng: column sets of
// the block's vectors, 1 or more)
MKPW_HD constexpr int dense_steps_ahead(int ng, int rt) { return ng * rt <= 2 ? 4 : ng * rt <= 4 ? 2 : 1; }

// Entries of the table of column offsets: whole chunks, and the lookahead past the
// last one, the next step's entry among them (4 (ahead + 1) columns, 20 at most)
MKPW_HD constexpr int dense_ncol(int kc, int npwx) { return (npwx + kc - 1) / kc * kc + 64; }

// LDS of a workgroup in bytes: the box, staged psi, D, the column offsets, the
// vector list; after the sum over G the projector sums, lambda and gamma, then
// the output tiles, take the place of the box and of psi
struct DenseLds {
  size_t buf, dl, wcol, slot, bytes;
};
MKPW_HD constexpr DenseLds dense_lds(int real, int nw, int ngm, int rt, int npwx, int nhalf, int nproj, int nall) {
  const size_t cs = 2 * (size_t)real, nb = 8 * (size_t)ngm;
  const size_t box = ((size_t)nhalf * cs + 15) / 16 * 16, buf = 2 * nb * dense_bs(nw, ngm, rt, real) * real;
  const size_t proj = nall > 0 ? ((size_t)nw * 16 + 16 + kDenseGS) * nb * cs : 0,
               tile = (size_t)nw * nb * kDenseTS * cs;
  size_t work = box + buf;
  if (proj > work) work = proj;
  if (tile > work) work = tile;
  DenseLds L{};
  L.buf = box;
  L.dl = work;
  L.wcol = L.dl + (size_t)nproj * nproj * cs;
  L.slot = L.wcol + sizeof(int) * (size_t)dense_ncol(dense_kc(nw, ngm, rt), npwx);
  L.bytes = L.slot + sizeof(int) * (nb + 4);
  return L;
}

// Waves of a workgroup, groups of 8 vectors and row tiles of a wave; vector blocks
// and row splits per k
struct DenseShape {
  int nw, ngm, rt, nbt, nsplit;
};

// Time of a launch in us: a start, then the rounds of workgroups of a CU (one of
// eight waves at a time, or two of four where both fit its LDS; one of four alone
// takes somewhat more than half), each the copy of its box, its projectors and, for
// every row tile of a wave and plane wave, the products of the block's vectors (sets
// of two in FP64, groups of eight in complex64).  Fitted to 4600 timed launches of
// 128 to 1200 k, 5 to 32 vectors and 130 to 930 plane waves: nine in ten within 15%.
inline double dense_us(int real, const DenseShape& s, int nk, int nvec, int npwmax, int npwx, int nhalf, int nproj,
                       int nall) {
  const long m = ((long)nk * s.nbt * s.nsplit + kDenseCus - 1) / kDenseCus;  // workgroups of the fullest CU
  const bool two = s.nw == 4 && 2 * dense_lds(real, s.nw, s.ngm, s.rt, npwx, nhalf, nproj, nall).bytes <= kDenseLdsPerCu;
  const double rounds = s.nw == 8 ? (double)m : two ? m / 2 + 0.62 * (m % 2) : 0.62 * m;
  const int kc = dense_kc(s.nw, s.ngm, s.rt), nb = std::min(nvec, 8 * s.ngm);
  const double work = (double)s.rt * ((npwmax + kc - 1) / kc * kc), sets = real == 8 ? (nb + 1) / 2 : (nb + 7) / 8;
  if (real == 8)
    return 4.6 + rounds * (1.33e-4 * 16 * nhalf + 0.66 * nall + (s.nw == 8 ? 0.0076 * sets * work
                                                                             : 3.1 + 0.0084 * sets * work));
  return 7.2 + rounds * (3.0e-4 * 8 * nhalf + 0.25 * nall + (0.0163 * sets + 0.0005) * work);
}

// Time of the transforms in us: the lines of the three passes over an n^3 mesh with
// a window of w, and the projectors (same launches, nine in ten within 10%)
inline double transforms_us(int real, int n, int w, long rows, int npwmax, int nproj) {
  const double lines = n * std::log2((double)n) * (0.79 * w * w + (double)w * n + (double)n * n);
  return real == 8 ? 13.5 + 1e-6 * rows * (0.3726 * lines + 3.6 * nproj * npwmax)
                   : 10.6 + 1e-6 * rows * (0.174 * lines + 1.74 * nproj * npwmax);
}

inline DenseShape dense_shape(int real, int nk, int nvec, int npwmax, int npwx, int nhalf, int nproj, int nall) {
  const bool fp64 = real == 8;
  const int groups = (nvec + 7) / 8;
  const int tiles = std::max(1, (npwmax + 15) / 16);
  auto lds = [&](int nw, int ngm, int rt) { return dense_lds(real, nw, ngm, rt, npwx, nhalf, nproj, nall).bytes; };
  // as many vectors per workgroup as fit (each entry of the box that is read
  // serves them all); two workgroups of four waves per CU where two fit, else
  // one of eight
  int ngm = std::min(3, groups);
  while (ngm > 1 && lds(8, ngm, 4) > kDenseLdsPerCu) --ngm;
  int nbt = (groups + ngm - 1) / ngm;
  const int nw = lds(4, ngm, 4) * 2 <= kDenseLdsPerCu ? 4 : 8;
  const int rmax = nw == 8 ? 4 : fp64 ? (ngm == 3 ? 5 : 6) : 8;
  const int least = (tiles + nw * rmax - 1) / (nw * rmax), most = std::max(least, (tiles + nw - 1) / nw);
  // a launch that leaves the chip part empty whatever its rows takes fewer vectors
  // per workgroup
  const long fill = kDenseCus * (8 / nw);
  while ((long)nk * nbt * most < fill && nbt < groups) ++nbt;
  ngm = (groups + nbt - 1) / nbt;
  // the row split of the least time: more rows to a workgroup share the box and the
  // projectors, fewer fill the chip and its last round
  DenseShape best{};
  double least_us = 0.0;
  for (int nsplit = least; nsplit <= most; ++nsplit) {
    DenseShape s{nw, ngm, (tiles + nsplit * nw - 1) / (nsplit * nw), nbt, nsplit};
    if (lds(nw, ngm, s.rt) > kDenseLdsPerCu) s.rt = 3;  // the smaller staging of larger blocks
    const double us = dense_us(real, s, nk, nvec, npwmax, npwx, nhalf, nproj, nall);
    if (nsplit == least || us < least_us) {
      best = s;
      least_us = us;
    }
  }
  return best;
}

// Whether the dense product of nvec vectors at nk k-points takes less time than the
// transforms on an n^3 mesh with a window of w.  By size, us (transforms / dense):
//   * up to 128 plane waves it is one short sum: 4 k x 5 vectors [110] 11.4 / 12.3, 1000
//     k x 24 [115] 230 / 82;
//   * up to 160, and in FP64 up to 368 with 512 k or more, it is the faster or within
//     3 us: 260 k x 6 [149] 29 / 25 (complex64 16 / 19), 600 k x 6 [363] 119 / 118;
//   * beyond, the sum grows as npw^2 and has to fill whole rounds of the CUs, and the
//     transforms grow with the mesh: FP64, 512 k x 16, 4 projectors [394, 20^3] 265 /
//     219, [571, 24^3] 405 / 431, [648, 24^3] 412 / 572, [728, 30^3] 712 / 647; with 16
//     projectors [648] 703 / 601: the two estimates are compared;
//   * few vectors share each entry of the box too little, and few k leave the chip
//     part empty: 1200 k x 3 [363] 132 / 155, 90 k x 10 [290] 50 / 78;
//   * complex64 sums of more than 520 terms are left to the transforms, whose rounding
//     does not grow with the basis.
inline bool dense_faster(int real, int nk, int nvec, int npwmax, int npwx, int nhalf, int nproj, int nall, int n,
                         int w) {
  if (npwmax <= 128) return nvec >= 3;
  if (nvec < 6 || nk < 256) return false;
  if (real != 8 && npwmax > 520) return false;
  if (npwmax <= 160 || (real == 8 && npwmax <= 368 && nk >= 512)) return true;
  const DenseShape s = dense_shape(real, nk, nvec, npwmax, npwx, nhalf, nproj, nall);
  return dense_us(real, s, nk, nvec, npwmax, npwx, nhalf, nproj, nall) <
         0.97 * transforms_us(real, n, w, (long)nk * nvec, npwmax, nall);
}

}  // namespace mkpw
