"""H|psi> by the transforms in launches of a row per CU or fewer, which take a shape
of their own (the whole mesh as one slab where it fits), against the oracle's dense
H; and the next larger launch, which does not.  Bounds as for H|psi> elsewhere."""
import numpy as np
import pytest

from oracle import hamiltonian as ham
from paper_2412_01695_amd import synth

from gpu_util import torch_cuda
from test_gpu_hpsi import TOL32, TOL64, _compare, _oracle_rows, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ecut,mesh,nproj", [(24.0, 18, 17), (32.0, 20, 24), (40.0, 24, 4), (48.0, 24, 24), (50.0, 36, 18)])
def test_few_rows(ecut, mesh, nproj):
    torch = torch_cuda()
    from paper_2412_01695_amd import mkpw
    from paper_2412_01695_amd.system import System
    c = synth.make_config(3)
    rng = np.random.default_rng([int(ecut), nproj])
    k = rng.uniform(-0.5, 0.5, (16, 3)) @ synth.reciprocal_rows(c.lat)
    proj = synth._sp_projectors([0, 1], [1.0, 1.3, 1.6])[:nproj]
    d = rng.standard_normal((nproj, nproj)) + 1j * rng.standard_normal((nproj, nproj))
    cfg = synth.Config(f"few-{ecut:g}", c.lat, ecut, (mesh,) * 3, k, 17, c.tau, proj, 0.1 * (d + d.conj().T), 7)
    s = System(cfg, 0, vloc=np.random.default_rng(8).standard_normal(cfg.fft))
    ks = [0, 7, 15]
    shapes = []
    for nb in (1, 16, 17):  # 16, 256 and 272 rows
        psi = s.psi_guess(nb)
        ref = _oracle_rows(cfg, s, ham.vtilde(s.vloc), psi, ks)
        for prec, tol in ((0, TOL64), (1, TOL32)):
            _compare(_run(torch, s, psi, prec), ref, s, tol)
            shapes.append([mkpw.pw_get_option(s.ctx, f"hpsi_{a}_tuned") for a in ("variant", "slab", "threads")])
    print(cfg.name, s.npwx, shapes)
    assert shapes[:2] == shapes[2:4] and all(v[0] != 6 for v in shapes)
