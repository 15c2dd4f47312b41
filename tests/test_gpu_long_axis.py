"""Response calls on a mesh that the library chooses, with one axis of more points
than any mesh it accepts as given (512): a cell long along one vector.

Bounds as for the same calls elsewhere: 1e-12 of the largest value of the
oracle's result."""
import numpy as np
import pytest

from oracle import dft, response
from paper_2412_01695_amd import synth

from gpu_util import to_dev, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("axis,length", [(0, 160.0), (1, 215.0)])
def test_long_axis(axis, length):
    torch = torch_cuda()
    from paper_2412_01695_amd import mkpw
    ecut, nk, nb = 30.0, 2, 2
    lat = np.diag([2.6, 2.6, 2.6])
    lat[axis, axis] = length
    rng = np.random.default_rng(axis)
    kpts = rng.uniform(-0.5, 0.5, (nk, 3)) @ synth.reciprocal_rows(lat)
    ctxs, npws, millers, npwxs = [], [], [], []
    for kk in (kpts, kpts + np.array([0.1, -0.2, 0.15])):
        ctx = mkpw.pw_create(0)
        mkpw.pw_set_lattice(ctx, lat)
        mkpw.pw_set_cutoff(ctx, ecut)
        npw, npwx = mkpw.pw_set_kpoints(ctx, kk)
        ctxs.append(ctx)
        npws.append(npw)
        npwxs.append(npwx)
        millers.append([mkpw.pw_get_miller(ctx, ik) for ik in range(nk)])
    try:
        ck, cq = ctxs
        fft = tuple(mkpw.pw_get_option(ck, f"fft{a}") for a in (1, 2, 3))
        assert max(fft) > 512
        dv = rng.standard_normal(fft) + 1j * rng.standard_normal(fft)
        dvt = dft.forward(dv)
        uk = np.zeros((nk, nb, npwxs[0]), complex)
        uq, du, ref = (np.zeros((nk, nb, npwxs[1]), complex) for _ in range(3))
        for ik in range(nk):
            n, m = int(npws[0][ik]), int(npws[1][ik])
            uk[ik, :, :n] = rng.standard_normal((nb, n)) + 1j * rng.standard_normal((nb, n))
            du[ik, :, :m] = rng.standard_normal((nb, m)) + 1j * rng.standard_normal((nb, m))
            v = np.linalg.qr(rng.standard_normal((m, nb)) + 1j * rng.standard_normal((m, nb)))[0]
            uq[ik, :, :m] = v.T
            dvu = response.dv_cross_matrix(millers[1][ik], millers[0][ik], fft, dvt) @ uk[ik, :, :n].T
            ref[ik, :, :m] = response.dfpt_rhs_q(dvu, v, None).T
        d_uk, d_uq, d_du = (to_dev(torch, a) for a in (uk, uq, du))
        out = torch.full((nk, nb, npwxs[1]), float("nan"), dtype=torch.complex128, device="cuda")
        torch.cuda.synchronize()
        mkpw.pw_dfpt_rhs(cq, ck, nb, dv, d_uk, d_uq, out)
        torch.cuda.synchronize()
        err = np.max(np.abs(out.cpu().numpy() - ref)) / np.max(np.abs(ref))
        print(fft, "rhs rel err", err)
        assert err <= 1e-12
        w = np.array([0.4, 0.6])
        ref = response.drho(fft, w, millers[0], [uk[ik, :, :npws[0][ik]] for ik in range(nk)],
                            millers[1], [du[ik, :, :npws[1][ik]] for ik in range(nk)])
        out = torch.full(fft, float("nan"), dtype=torch.complex128, device="cuda")
        torch.cuda.synchronize()
        mkpw.pw_drho(cq, ck, nb, w, d_uk, d_du, out)
        torch.cuda.synchronize()
        err = np.max(np.abs(out.cpu().numpy() - ref)) / np.max(np.abs(ref))
        print(fft, "drho rel err", err)
        assert err <= 1e-12
    finally:
        for ctx in ctxs:
            mkpw.pw_destroy(ctx)
