// Launch shapes of the dense H|psi> product (hpsi_dense.hip) and the ranges of its
// LDS and of psi that a shape reads.  Plain arithmetic, so that a host program can
// walk every shape without a GPU.
#pragma once

#include <algorithm>
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
  int nsplit = (tiles + nw * rmax - 1) / (nw * rmax);
  // a launch that leaves the chip part empty takes fewer rows per workgroup,
  // then fewer vectors
  const long fill = kDenseCus * (8 / nw);
  while ((long)nk * nbt * nsplit < fill && nsplit * nw < tiles) ++nsplit;
  while ((long)nk * nbt * nsplit < fill && nbt < groups) ++nbt;
  ngm = (groups + nbt - 1) / nbt;
  int rt = (tiles + nsplit * nw - 1) / (nsplit * nw);
  if (lds(nw, ngm, rt) > kDenseLdsPerCu) rt = 3;  // the smaller staging of larger blocks
  return {nw, ngm, rt, nbt, nsplit};
}

}  // namespace mkpw
