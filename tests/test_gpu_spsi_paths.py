"""S|psi> at the sizes where one of its kernels hands over to another: projector and
row counts on both sides of each limit, few and many k-points, with rows left out
of the selection in place.  Against the sums of the definition in double precision;
bounds as for S|psi> elsewhere, 1e-13 (FP64) and 2e-6 (complex64) of the largest
element."""
import numpy as np
import pytest

from paper_2412_01695_amd import synth

from gpu_util import to_dev, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ecut,nk", [(6.0, 300), (24.0, 270), (30.0, 270), (36.0, 270), (42.0, 262), (62.0, 258),
                                     (30.0, 40), (62.0, 520)])
def test_on_both_sides_of_each_limit(ecut, nk):
    torch = torch_cuda()
    from paper_2412_01695_amd import mkpw
    c = synth.make_config(1)
    rng = np.random.default_rng([int(ecut), nk])
    ctx = mkpw.pw_create(0)
    try:
        mkpw.pw_set_lattice(ctx, c.lat)
        mkpw.pw_set_cutoff(ctx, ecut, (36,) * 3)
        npw, npwx = mkpw.pw_set_kpoints(ctx, rng.uniform(-0.5, 0.5, (nk, 3)) @ synth.reciprocal_rows(c.lat))
        ok = torch.from_numpy(np.arange(npwx)[None] < npw[:, None]).cuda()
        for nproj in (2, 3, 4, 5, 7, 8, 9, 12, 13):
            beta = rng.standard_normal((nk, nproj, npwx, 2)).view(complex)[..., 0]
            beta /= np.sqrt(npwx)
            q = rng.standard_normal((nproj, nproj)) + 1j * rng.standard_normal((nproj, nproj))
            q = 0.2 * (q + q.conj().T)
            mkpw.pw_set_projectors(ctx, beta, np.eye(nproj) + 0j)
            mkpw.pw_set_qij(ctx, q)
            b = torch.where(ok[:, None], to_dev(torch, beta), 0)
            for nb in (1, 3, 4, 9):
                psi = torch.where(ok[:, None], torch.randn(nk, nb, npwx, dtype=torch.complex128, device="cuda"), 0)
                ref = psi.clone()
                lam = (b.conj()[:, :, None] * psi[:, None]).sum(-1)  # (nk, nproj, nb)
                delta = (to_dev(torch, q)[None, :, :, None] * lam[:, None]).sum(2)
                for p in range(nproj):
                    ref += delta[:, p, :, None] * b[:, p, None]
                dirty = torch.where(ok[:, None], psi, float("nan"))  # what the padding holds is not read
                for prec, dt, tol in ((0, torch.complex128, 1e-13), (1, torch.complex64, 2e-6)):
                    x = dirty.to(dt, copy=True)
                    out = torch.full_like(x, float("nan"))
                    torch.cuda.synchronize()
                    mkpw.pw_s_psi(ctx, prec, nb, x, out)
                    mkpw.pw_s_psi(ctx, prec, nb, x, x)
                    torch.cuda.synchronize()
                    for got in (out, x):
                        err = float((got.to(torch.complex128) - ref).abs().max() / ref.abs().max())
                        assert err <= tol, (npwx, nproj, nb, prec, err)
    finally:
        mkpw.pw_destroy(ctx)
