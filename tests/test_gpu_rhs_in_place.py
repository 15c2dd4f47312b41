"""Response right-hand sides written over the states they are formed from: the same
result as in an array of their own, where a k-point's rows and bands are shared out
over workgroups that read them while others write, and where the right-hand sides of
one k-point land on the states of one that is taken later."""
import numpy as np
import pytest

from paper_2412_01695_amd import synth

from gpu_util import to_dev, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nk,ecut,nocc,shift", [(2, 30.0, 16, 0), (300, 9.0, 9, 0), (300, 30.0, 8, 3000)])
def test_over_its_input(nk, ecut, nocc, shift):
    torch = torch_cuda()
    from paper_2412_01695_amd import mkpw
    from paper_2412_01695_amd.system import System
    c = synth.make_config(1)
    rng = np.random.default_rng([nk, nocc])
    kpts = rng.uniform(-0.5, 0.5, (nk, 3)) @ synth.reciprocal_rows(c.lat)
    cfg = synth.Config(f"rhs-in-place-{nk}", c.lat, ecut, (36 if ecut > 16 else 15,) * 3, kpts, nocc, c.tau,
                       c.projectors, c.dij, 9)
    sk, sq = System(cfg, 0), System(synth.shifted(cfg, synth.q_paper()), 0)
    assert sk.npwx == sq.npwx
    dv = synth.dv_complex_grid(cfg)
    size = nk * nocc * sk.npwx
    u = to_dev(torch, rng.standard_normal((size, 2)).view(complex)[:, 0])
    shape = (nk, nocc, sk.npwx)
    occ = to_dev(torch, np.linalg.qr(rng.standard_normal((nk, sk.npwx, nocc)))[0].transpose(0, 2, 1) + 0j)
    ref = torch.empty(shape, dtype=torch.complex128, device="cuda")
    buf = torch.zeros(size + shift, dtype=torch.complex128, device="cuda")
    buf[:size] = u
    torch.cuda.synchronize()
    mkpw.pw_dfpt_rhs(sq.ctx, sk.ctx, nocc, dv, u.view(shape), occ, ref)
    mkpw.pw_dfpt_rhs(sq.ctx, sk.ctx, nocc, dv, buf[:size].view(shape), occ, buf[shift:].view(shape))
    torch.cuda.synchronize()
    got = buf[shift:].view(shape)
    # the sum over the k sphere may be grouped otherwise: each within the oracle's bound
    assert float((got - ref).abs().max()) <= 2e-12 * float(ref.abs().max())
