"""Density response where a workgroup sums several k-points: each k is summed by
itself first.

One k repeated, every pair product the same value c = 1 + 2^-44 - 2^-52: adding c
to a sum of 512 or more loses 2^-44 (almost half a unit in the last place) every
time, and to a smaller one next to nothing.  A k has at most npw < 512 pairs in a
bin, so k by k the sums are good to rounding; one running sum over a workgroup's 32
k-points is 4e-14 short.  Bound: one rounding for each addition that follows, 32 k
of a workgroup, 8 boxes of a chunk, 32 chunks and three axes of 20 points,
132 x 2^-53 = 1.5e-14 of the largest value (all terms are positive)."""
import numpy as np
import pytest

from paper_2412_01695_amd import synth

from gpu_util import to_dev, torch_cuda
from test_gpu_drho_units import test_drho_shares as _shares

pytestmark = pytest.mark.gpu


def test_each_k_summed_by_itself():
    torch = torch_cuda()
    from paper_2412_01695_amd import mkpw
    nk, n = 8192, 20
    c = synth.make_config(1)
    kpts = np.tile([0.01, 0.02, 0.03], (nk, 1))
    ctxs = []
    for _ in range(2):
        ctx = mkpw.pw_create(0)
        mkpw.pw_set_lattice(ctx, c.lat)
        mkpw.pw_set_cutoff(ctx, 30.0, (n,) * 3)
        npw, npwx = mkpw.pw_set_kpoints(ctx, kpts)
        ctxs.append(ctx)
    try:
        m = mkpw.pw_get_miller(ctxs[0], 0)
        assert 256 < len(m) < 512
        val = 1.0 + 2.0**-44 - 2.0**-52  # 4 w conj(u) du, exact
        row = np.zeros(npwx, complex)
        row[:len(m)] = 1.0
        d_u = to_dev(torch, row).expand(nk, 1, npwx).contiguous()
        d_du = d_u * (val / 4.0)
        out = torch.full((n,) * 3, float("nan"), dtype=torch.complex128, device="cuda")
        torch.cuda.synchronize()
        mkpw.pw_drho(ctxs[1], ctxs[0], 1, np.ones(nk), d_u, d_du, out)
        torch.cuda.synchronize()
    finally:
        for ctx in ctxs:
            mkpw.pw_destroy(ctx)
    count = np.zeros((n,) * 3)  # pairs per Miller difference
    d = (m[None] - m[:, None]).reshape(-1, 3) % n
    np.add.at(count, tuple(d.T), 1.0)
    ref = np.fft.ifftn(count * nk) * n**3 * val
    err = np.max(np.abs(out.cpu().numpy() - ref)) / np.max(np.abs(ref))
    print("drho rel err", err)
    assert err <= 132 * 2.0**-53


@pytest.mark.parametrize("nk,ecut,nb", [(300, 4.0, 9), (520, 3.0, 17)])
def test_several_k_per_workgroup_by_band_count(nk, ecut, nb):
    # the kernels of 9 to 16 bands and of more
    _shares(nk, ecut, nb, 0)
