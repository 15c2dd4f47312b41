"""DFPT CG at every row length its update kernel is built for (one wave per
system up to 512 plane waves, four to 2048, the two kernels apart beyond), with
the valence projector inside the H|psi> product (up to 16 projectors and
occupied bands together) and beside it: the third iterate against the oracle's
recurrence.

Bound 1e-10 of the largest element, as for the third iterate elsewhere: three
updates amplify rounding (1e-15 of ||A|| ||x||) by the few orders the
preconditioned systems' condition gives."""
import numpy as np
import pytest

from oracle import hamiltonian as ham, solvers
from paper_2412_01695_amd import synth

from gpu_util import to_dev, torch_cuda
from helpers import beta_fn, miller_map

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ecut,nocc,overlap", [
    (4.0, 3, False), (15.0, 4, False), (15.0, 12, True), (15.0, 13, False),  # folded up to 16 in all
    (20.0, 3, True), (27.0, 4, False), (33.0, 3, False), (37.0, 3, False), (42.0, 5, False),  # 3 .. 8 per lane
    (46.0, 3, False), (60.0, 3, True), (72.0, 3, False), (95.0, 3, False), (112.0, 2, False)])
def test_third_iterate(ecut, nocc, overlap):
    torch = torch_cuda()
    from paper_2412_01695_amd import mkpw
    from paper_2412_01695_amd.system import System
    c = synth.make_config(1)
    mesh = 15 if ecut < 20 else 36
    cfg = synth.Config(f"cg-{ecut:g}", c.lat, ecut, (mesh,) * 3, c.kpts[2:4], nocc, c.tau, c.projectors, c.dij, 9)
    if overlap:
        cfg = synth.with_overlap(cfg)
    s = System(cfg, 0)
    vt = ham.vtilde(s.vloc)
    rng = np.random.default_rng(int(ecut))
    u_l = np.zeros((cfg.nk, nocc, s.npwx), complex)
    rhs_l = np.zeros_like(u_l)
    eps = np.zeros((cfg.nk, nocc))
    ref = []
    for ik in range(cfg.nk):
        kp = ham.KPoint(cfg, ik, vt, beta_fn)
        n = kp.npw
        perm = miller_map(s.miller[ik], kp.miller)
        fall = 1.0 / (1.0 + kp.kin)[:, None]
        u = np.linalg.qr((rng.standard_normal((n, nocc)) + 1j * rng.standard_normal((n, nocc))) * fall)[0]
        b = (rng.standard_normal((n, nocc)) + 1j * rng.standard_normal((n, nocc))) * fall
        eps[ik] = -1.0 - 0.1 * np.arange(nocc)  # below the spectrum: positive definite
        u_l[ik, :, :n] = u.T[:, perm]
        rhs_l[ik, :, :n] = b.T[:, perm]
        for nu in range(nocc):
            a = solvers.dfpt_matrix(kp.h, u, eps[ik, nu], 0.7, kp.s if overlap else None)
            m = solvers.dfpt_precond(kp.kin, u[:, nu])
            x, _, _ = solvers.pcg(lambda v: a @ v, lambda v: v / m, b[:, nu], np.zeros(n), 1e-60, max_iter=3)
            ref.append(x[perm])
    du, drhs = to_dev(torch, u_l), to_dev(torch, rhs_l)
    dx = torch.zeros_like(drhs)
    torch.cuda.synchronize()
    st, _ = mkpw.pw_dfpt_cg(s.ctx, 0, nocc, du, eps, np.full(cfg.nk, 0.7), nocc, drhs, dx, 1e-60, 3)
    torch.cuda.synchronize()
    assert st == mkpw.PW_ENOCONV
    x = dx.cpu().numpy().reshape(cfg.nk * nocc, s.npwx)
    scale = max(np.max(np.abs(r)) for r in ref)
    for row, r, n in zip(x, ref, np.repeat(s.npw, nocc)):
        assert np.max(np.abs(row[:n] - r)) <= 1e-10 * scale
        assert np.all(row[n:] == 0)
