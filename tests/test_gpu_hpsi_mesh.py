"""H|psi> on the smaller mesh that the autotuned launches use (the one that
holds the Miller differences of the window) against the oracle's dense H on the
context's mesh.

The potential is white noise on the context's mesh, so every Fourier
coefficient is as large as the others and one that is dropped or wrapped wrongly
shows.  Bounds as for H|psi> elsewhere: 1e-13 (FP64) and 2e-6 (complex64) of the
largest element."""
import numpy as np
import pytest

from oracle import hamiltonian as ham
from paper_2412_01695_amd import synth

from gpu_util import torch_cuda
from test_gpu_hpsi import TOL32, TOL64, _compare, _oracle_rows, _run

pytestmark = pytest.mark.gpu


def _config(ecut, mesh, nk=5, nbnd=3):
    c = synth.make_config(1)
    k = np.random.default_rng(int(10 * ecut) + mesh).uniform(-0.5, 0.5, (nk, 3)) @ synth.reciprocal_rows(c.lat)
    return synth.Config(f"noise-{ecut:g}-{mesh}", c.lat, ecut, (mesh,) * 3, k, nbnd, c.tau, c.projectors, c.dij, 5)


def _noise(mesh, seed):
    return np.random.default_rng(seed).standard_normal((mesh,) * 3)


# windows of 6 to 11 on meshes from just enough (no smaller one) to 36^3
@pytest.mark.parametrize("ecut,mesh", [(8.0, 15), (12.0, 20), (15.0, 36), (25.0, 24), (30.0, 20), (30.0, 30),
                                       (40.0, 32), (40.0, 36)])
def test_white_noise_potential(ecut, mesh):
    torch = torch_cuda()
    from paper_2412_01695_amd.system import System
    cfg = _config(ecut, mesh)
    s = System(cfg, 0, vloc=_noise(mesh, 3))
    psi = s.psi_guess()
    ref = _oracle_rows(cfg, s, ham.vtilde(s.vloc), psi, range(cfg.nk))
    for prec, tol in ((0, TOL64), (1, TOL32)):
        _compare(_run(torch, s, psi, prec), ref, s, tol)


def test_new_potential_new_k_list_and_explicit_shapes_on_one_context():
    # what is kept of the potential follows each change, also when launches on
    # the context's own mesh (an explicit shape) come in between
    torch = torch_cuda()
    from paper_2412_01695_amd import mkpw
    from paper_2412_01695_amd.system import System
    cfg = _config(30.0, 36)
    s = System(cfg, 0, vloc=_noise(36, 4))
    psi = s.psi_guess()

    def check(variants):
        ref = _oracle_rows(s.cfg, s, ham.vtilde(s.vloc), psi, range(s.cfg.nk))
        for v in variants:
            mkpw.pw_set_option(s.ctx, "hpsi_variant", v)
            _compare(_run(torch, s, psi, 0), ref, s, TOL64)
        mkpw.pw_set_option(s.ctx, "hpsi_variant", 0)

    check((0, 4, 0, 1, 0))
    s.vloc = _noise(36, 5)
    mkpw.pw_set_vloc(s.ctx, s.vloc)
    check((0, 1, 4, 0))
    # another k-list (no projectors: setting k-points removes them)
    s.cfg = cfg = synth.Config("noise-2", cfg.lat, cfg.ecut_ry, cfg.fft, cfg.kpts[::-1] * 0.7, 3, cfg.tau, [],
                               np.zeros((0, 0), complex), 6)
    s.npw, s.npwx = mkpw.pw_set_kpoints(s.ctx, cfg.kpts)
    s.miller = [mkpw.pw_get_miller(s.ctx, ik, int(n)) for ik, n in enumerate(s.npw)]
    psi = s.psi_guess()
    check((0, 4, 0))
