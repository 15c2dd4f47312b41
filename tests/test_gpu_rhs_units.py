"""Response right-hand sides over the ways the pair product is shared out: the
box of Miller differences in LDS with units of several k-points per workgroup, a
k-point's rows split over workgroups, both block lengths, band counts around the
groups of 8 and 16, more row tiles than one unit holds, and the box read from
memory where it does not fit.

Bound 1e-12 of the largest element of the oracle's result, as for the same
product elsewhere."""
import numpy as np
import pytest

from oracle import dft, hamiltonian as ham, response
from paper_2412_01695_amd import synth

from gpu_util import to_dev, torch_cuda
from helpers import beta_fn, miller_map

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nk,ecut,nocc", [
    (1, 30.0, 8), (2, 9.0, 9), (300, 4.0, 3), (270, 6.0, 16), (3, 12.0, 17), (2, 22.0, 1), (2, 35.0, 7),
    (2, 38.5, 20), (2, 44.0, 9)])
def test_rhs_shares(nk, ecut, nocc):
    torch = torch_cuda()
    from paper_2412_01695_amd import mkpw
    from paper_2412_01695_amd.system import System
    c = synth.make_config(1)
    rng = np.random.default_rng([nk, int(ecut), nocc])
    mesh = 15 if ecut < 16 else 36
    kpts = rng.uniform(-0.5, 0.5, (nk, 3)) @ synth.reciprocal_rows(c.lat)
    cfg = synth.Config(f"rhs-{nk}", c.lat, ecut, (mesh,) * 3, kpts, nocc, c.tau, c.projectors, c.dij, 9)
    sk, sq = System(cfg, 0), System(synth.shifted(cfg, synth.q_paper()), 0)
    dv = synth.dv_complex_grid(cfg)
    dvt = dft.forward(dv)
    vt = ham.vtilde(sk.vloc)
    uk = np.full((nk, nocc, sk.npwx), np.nan, complex)  # what the padding holds is not read
    uq = np.zeros((nk, nocc, sq.npwx), complex)
    ref = np.zeros_like(uq)
    for ik in range(nk):
        kk, kq = ham.KPoint(cfg, ik, vt, beta_fn), ham.KPoint(sq.cfg, ik, vt, beta_fn)
        pk, pq = miller_map(sk.miller[ik], kk.miller), miller_map(sq.miller[ik], kq.miller)
        a = rng.standard_normal((2, kk.npw, nocc)) @ np.diag(np.ones(nocc))
        u = a[0] + 1j * a[1]
        v = np.linalg.qr(rng.standard_normal((kq.npw, nocc)) + 1j * rng.standard_normal((kq.npw, nocc)))[0]
        r = response.dfpt_rhs_q(response.dv_cross_matrix(kq.miller, kk.miller, cfg.fft, dvt) @ u, v, None)
        uk[ik, :, :kk.npw], uq[ik, :, :kq.npw], ref[ik, :, :kq.npw] = u.T[:, pk], v.T[:, pq], r.T[:, pq]
    d_uk, d_uq = to_dev(torch, uk), to_dev(torch, uq)
    out = torch.full((nk, nocc, sq.npwx), float("nan"), dtype=torch.complex128, device="cuda")
    torch.cuda.synchronize()
    mkpw.pw_dfpt_rhs(sq.ctx, sk.ctx, nocc, dv, d_uk, d_uq, out)
    torch.cuda.synchronize()
    err = np.max(np.abs(out.cpu().numpy() - ref)) / np.max(np.abs(ref))
    print("nk", nk, "npwx", sk.npwx, "rhs rel err", err)
    assert err <= 1e-12
