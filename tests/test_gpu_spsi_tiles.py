"""S|psi> on the matrix cores against the oracle's dense S where its tiles end:
rows of 1 to 16 tiles a wave, projector counts around its two tile shapes and
past them, band counts around its groups of eight, in and out of place.

Bounds as for S|psi> elsewhere: 1e-13 (FP64) and 2e-6 (complex64) of the largest
element."""
import numpy as np
import pytest

from oracle import hamiltonian as ham
from paper_2412_01695_amd import synth

from gpu_util import to_dev, torch_cuda
from helpers import beta_fn, miller_map

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ecut,nbnd,nproj", [
    (3.0, 1, 1), (6.0, 7, 8), (12.0, 8, 9), (16.0, 9, 16), (22.0, 17, 7), (27.0, 3, 16), (33.0, 16, 8),
    (37.0, 5, 12), (43.0, 8, 3), (52.0, 2, 8), (62.0, 9, 16), (15.0, 5, 17), (70.0, 3, 8), (15.0, 4, 24)])
def test_tile_edges(ecut, nbnd, nproj):
    torch = torch_cuda()
    from paper_2412_01695_amd import mkpw
    from paper_2412_01695_amd.system import System
    c = synth.make_config(3)
    rng = np.random.default_rng([int(ecut), nbnd, nproj])
    mesh = 15 if ecut < 17 else 36
    k = rng.uniform(-0.5, 0.5, (3, 3)) @ synth.reciprocal_rows(c.lat)
    proj = synth._sp_projectors([0, 1], [1.0, 1.3, 1.6])[:nproj]
    d, q = (m + m.conj().T for m in rng.standard_normal((2, nproj, nproj)) + 1j * rng.standard_normal((2, nproj, nproj)))
    cfg = synth.with_overlap(synth.Config(f"spsi-{ecut:g}", c.lat, ecut, (mesh,) * 3, k, nbnd, c.tau, proj, d, 7), 0.2 * q)
    s = System(cfg, 0)
    vt = ham.vtilde(s.vloc)
    psi = np.full((cfg.nk, nbnd, s.npwx), np.nan, complex)  # what the padding holds is not read
    ref = np.zeros_like(psi)
    for ik in range(cfg.nk):
        kp = ham.KPoint(cfg, ik, vt, beta_fn)
        perm = miller_map(s.miller[ik], kp.miller)
        v = rng.standard_normal((kp.npw, nbnd)) + 1j * rng.standard_normal((kp.npw, nbnd))
        psi[ik, :, :kp.npw] = v.T[:, perm]
        ref[ik, :, :kp.npw] = (kp.s @ v).T[:, perm]
    for prec, dt, tol in ((0, torch.complex128, 1e-13), (1, torch.complex64, 2e-6)):
        a = to_dev(torch, psi, dt)
        out = torch.full_like(a, float("nan"))
        torch.cuda.synchronize()
        mkpw.pw_s_psi(s.ctx, prec, nbnd, a, out)
        mkpw.pw_s_psi(s.ctx, prec, nbnd, a, a)
        torch.cuda.synchronize()
        for got in (out, a):
            err = np.max(np.abs(got.cpu().numpy() - ref)) / np.max(np.abs(ref))
            print("npwx", s.npwx, "prec", prec, "rel err", err)
            assert err <= tol
