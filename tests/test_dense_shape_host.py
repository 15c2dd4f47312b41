"""What the dense H|psi> product reads, over every launch shape it can take.

The shape rules and the index of a staged value are plain arithmetic in
csrc/hpsi_dense_shape.hpp; a host program walks them: no element of psi past its
row, no column offset past its table, every row and vector covered, and the LDS
within a CU's."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

WALK = r"""
#include <cstdio>
#include "hpsi_dense_shape.hpp"
using namespace mkpw;
int main() {
  long shapes = 0;
  for (int real : {4, 8})
    for (int npwx = 64; npwx <= 1280; npwx += 64)
      for (int npw : {npwx - 63, npwx - 48, npwx - 17, npwx - 1, npwx})
        for (int nk : {1, 2, 4, 31, 128, 255, 256, 300, 511, 512, 1024, 4096})
          for (int nvec = 1; nvec <= 50; ++nvec)
            for (int nhalf : {1, 172, 1331, 4631, 6084, 7813, 8900})
              for (int nproj : {0, 4, 16}) {
                if (dense_lds(8, 8, 1, 3, npwx, nhalf, 16, 16).bytes > kDenseLdsPerCu) continue;  // not taken
                const DenseShape s = dense_shape(real, nk, nvec, npw, npwx, nhalf, nproj, nproj);
                const int kc = dense_kc(s.nw, s.ngm, s.rt), nch = (npw + kc - 1) / kc;
                const char* bad = nullptr;
                for (int c = 0; c < nch; ++c)
                  for (int t = 0; t < kc; ++t) {
                    const int g = dense_psi_index(c, kc, t, npw);
                    if (g < 0 || g >= npwx) bad = "psi read past its row";
                    if (c * kc + t < npw && g != c * kc + t) bad = "another plane wave staged";
                  }
                // sets of a block: up to 4 per group of 8 vectors, 1 at least
                int ahead = 0;
                for (int ng = 1; ng <= 4 * s.ngm; ++ng)
                  if (dense_steps_ahead(ng, s.rt) > ahead) ahead = dense_steps_ahead(ng, s.rt);
                // the entry after the last step's lookahead, four columns to a step
                if (nch * kc + 4 * ahead + 3 >= dense_ncol(kc, npwx)) bad = "column offset past the table";
                const size_t lds = dense_lds(real, s.nw, s.ngm, s.rt, npwx, nhalf, nproj, nproj).bytes;
                if (lds > kDenseLdsPerCu) bad = "LDS";
                if (s.nsplit * s.nw * s.rt * 16 < npw) bad = "rows left out";
                if (s.nbt * s.ngm * 8 < nvec) bad = "vectors left out";
                if (s.ngm < 1 || s.ngm > 3 || s.rt < 1 || s.rt > (s.nw == 8 ? 4 : real == 8 ? 6 : 8)) bad = "no kernel";
                if (bad) {
                  std::printf("%s: real %d npwx %d npw %d nk %d nvec %d nhalf %d nproj %d (nw %d ngm %d rt %d)\n", bad,
                              real, npwx, npw, nk, nvec, nhalf, nproj, s.nw, s.ngm, s.rt);
                  return 1;
                }
                ++shapes;
              }
  std::printf("%ld shapes\n", shapes);
  return 0;
}
"""


# real, k, vectors, plane waves, window, projectors, mesh; us of the transforms and of
# the product.  Launches where one path takes more than the other by a sixth or more.
TIMED = [
    (8, 700, 16, 648, 12, 4, 24, 581, 842), (8, 512, 6, 648, 12, 4, 24, 160, 281), (8, 300, 12, 820, 13, 4, 30, 341, 471),
    (8, 400, 16, 696, 11, 4, 24, 319, 580), (8, 1000, 8, 696, 11, 4, 24, 415, 638), (8, 300, 6, 728, 13, 4, 30, 180, 231),
    (8, 512, 12, 928, 12, 16, 24, 606, 829), (8, 317, 6, 362, 10, 4, 20, 70, 101),
    (8, 512, 20, 316, 10, 8, 20, 334, 163), (8, 1728, 24, 490, 11, 4, 24, 1860, 1415), (8, 600, 24, 490, 11, 4, 24, 650, 545),
    (8, 400, 6, 173, 8, 4, 15, 38, 29), (8, 1000, 16, 728, 13, 16, 30, 2144, 1380), (8, 317, 13, 705, 13, 16, 30, 499, 439),
    (4, 1000, 6, 571, 12, 4, 24, 147, 267), (4, 1200, 10, 363, 10, 8, 20, 179, 216), (4, 600, 6, 490, 11, 4, 24, 90, 113),
    (4, 2048, 16, 316, 10, 8, 20, 461, 258), (4, 1728, 24, 490, 11, 4, 24, 902, 748), (4, 1024, 24, 409, 11, 8, 24, 379, 323),
]


def _run(tmp_path, text):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(text)
    subprocess.run([cxx, "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2412_01695_amd", "csrc"), str(src),
                    "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], capture_output=True, text=True)


def test_every_shape_reads_in_bounds(tmp_path):
    r = _run(tmp_path, WALK)
    assert r.returncode == 0, r.stdout


def test_the_faster_path_is_taken(tmp_path):
    calls = []
    for real, nk, nv, npw, w, nproj, mesh, _, _ in TIMED:
        npwx, nhalf = (npw + 63) // 64 * 64, ((2 * w - 1)**3 + 1) // 2
        calls.append(f'std::printf("%d ", (int)dense_faster({real}, {nk}, {nv}, {npw}, {npwx}, {nhalf}, {nproj}, {nproj}, '
                     f'{mesh}, {w}));')
    r = _run(tmp_path, "#include <cstdio>\n#include \"hpsi_dense_shape.hpp\"\nusing namespace mkpw;\nint main() {\n"
             + "\n".join(calls) + "\nreturn 0;\n}\n")
    assert r.returncode == 0
    for row, took in zip(TIMED, r.stdout.split(), strict=True):
        assert bool(int(took)) == (row[-1] < row[-2]), row
