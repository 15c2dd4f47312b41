"""H|psi> recorded by the caller, replayed after what changes the copies of the
potential that its kernels read: launches of an explicit shape on the context's own
mesh, and a new potential (with one launch after it, which fills the copies)."""
import numpy as np
import pytest

from paper_2412_01695_amd import synth

from gpu_util import to_dev, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ecut,mesh,nb,dense", [(30.0, 36, 1, False), (24.0, 36, 2, False), (13.0, 15, 5, True)])
@pytest.mark.parametrize("prec", [0, 1])
def test_replays(ecut, mesh, nb, dense, prec):
    torch = torch_cuda()
    from paper_2412_01695_amd import mkpw
    from paper_2412_01695_amd.system import System
    c = synth.make_config(1)
    rng = np.random.default_rng([int(ecut), nb])
    kpts = rng.uniform(-0.5, 0.5, (4, 3)) @ synth.reciprocal_rows(c.lat)
    cfg = synth.Config(f"recorded-{ecut:g}", c.lat, ecut, (mesh,) * 3, kpts, nb, c.tau, c.projectors, c.dij, 9)
    st = torch.cuda.Stream()
    s = System(cfg, 0, stream=st, vloc=rng.standard_normal(cfg.fft))
    dt = torch.complex128 if prec == 0 else torch.complex64
    psi, out, eager = to_dev(torch, s.psi_guess(), dt), None, None
    out, eager = torch.empty_like(psi), torch.empty_like(psi)

    def run(dst):
        torch.cuda.synchronize()
        mkpw.pw_h_psi(s.ctx, prec, nb, psi, dst)
        torch.cuda.synchronize()
        return dst.cpu().numpy()

    run(out)
    assert (mkpw.pw_get_option(s.ctx, "hpsi_variant_tuned") == 6) == dense
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        mkpw.pw_h_psi(s.ctx, prec, nb, psi, out)

    def replayed():
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        return out.cpu().numpy()

    ref = run(eager)
    assert np.array_equal(replayed(), ref)
    for variant in (4, 1, 4):
        mkpw.pw_set_option(s.ctx, "hpsi_variant", variant)
        run(eager)
        filler = [torch.full((1 << 18,), 7.0, device="cuda") for _ in range(4)]  # memory given back is taken again
        mkpw.pw_set_option(s.ctx, "hpsi_variant", 0)
        assert np.array_equal(replayed(), ref)
        del filler
    for seed in (1, 2):
        mkpw.pw_set_vloc(s.ctx, np.random.default_rng(seed).standard_normal(cfg.fft))
        new = run(eager)
        assert not np.array_equal(new, ref)
        assert np.array_equal(replayed(), new)
