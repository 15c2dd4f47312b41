"""Density response over the ways its pair sum is shared out: several k-points
per workgroup in one box of bins (more k than CUs, an uneven share), a k-point
split over workgroups (few k), a box in slices, and a box per k-point where the
two lists lie apart in Miller space by k-dependent reciprocal vectors.

Bound 1e-12 of the largest value of the oracle's density, as for the same sum
elsewhere: at most 64 x 512 products of order one per value in FP64."""
import numpy as np
import pytest

from oracle import response
from paper_2412_01695_amd import synth

from gpu_util import to_dev, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nk,ecut,nb,apart", [
    (1, 30.0, 6, 0), (3, 9.0, 12, 0), (301, 4.0, 5, 0), (700, 3.0, 3, 0), (2, 44.0, 9, 0),
    (2, 30.0, 6, 26), (270, 4.0, 2, 120), (3, 9.0, 17, 40)])
def test_drho_shares(nk, ecut, nb, apart):
    torch = torch_cuda()
    from paper_2412_01695_amd import mkpw
    from paper_2412_01695_amd.system import System
    c = synth.make_config(1)
    rng = np.random.default_rng(nk)
    rec = 2.0 * np.pi * np.linalg.inv(np.asarray(c.lat)).T  # rows b_i for rows a_i
    mesh = 15 if ecut < 20 else 36
    kpts = rng.uniform(-0.5, 0.5, (nk, 3)) @ rec
    cfg = synth.Config(f"drho-{nk}", c.lat, ecut, (mesh,) * 3, kpts, nb, c.tau, c.projectors, c.dij, 9)
    far = synth.shifted(cfg, synth.q_paper())
    far.kpts = far.kpts + (np.arange(nk) % 2 * apart)[:, None] * rec[0]
    sk, sq = System(cfg, 0), System(far, 0)
    uk = np.zeros((nk, nb, sk.npwx), complex)
    du = np.zeros((nk, nb, sq.npwx), complex)
    for ik in range(nk):
        uk[ik, :, :sk.npw[ik]] = synth.random_vectors(5, ik, sk.miller[ik], nb)
        du[ik, :, :sq.npw[ik]] = synth.random_vectors(9, ik, sq.miller[ik], nb)
    w = rng.uniform(0.5, 1.5, nk) / nk
    ref = response.drho(cfg.fft, w, sk.miller, [uk[ik, :, :sk.npw[ik]] for ik in range(nk)],
                        sq.miller, [du[ik, :, :sq.npw[ik]] for ik in range(nk)])
    d_uk, d_du = to_dev(torch, uk), to_dev(torch, du)
    d_out = torch.full(cfg.fft, float("nan"), dtype=torch.complex128, device="cuda")
    torch.cuda.synchronize()
    for _ in range(2):  # the second call on used workspaces
        mkpw.pw_drho(sq.ctx, sk.ctx, nb, w, d_uk, d_du, d_out)
        torch.cuda.synchronize()
        err = np.max(np.abs(d_out.cpu().numpy() - ref)) / np.max(np.abs(ref))
        print("nk", nk, "drho rel err", err)
        assert err <= 1e-12
