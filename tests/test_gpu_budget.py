"""Memory budgets that hold exactly what a call needs: what the library keeps or
takes to be faster must not make the call fail."""
import numpy as np
import pytest

from paper_2412_01695_amd import synth

from gpu_util import to_dev, torch_cuda
from test_gpu_hpsi import TOL64

pytestmark = pytest.mark.gpu


def _budgeted(cfg, budget=0):
    from paper_2412_01695_amd import mkpw
    ctx = mkpw.pw_create(0)
    mkpw.pw_set_option(ctx, "hbm_budget_bytes", budget)
    mkpw.pw_set_lattice(ctx, cfg.lat)
    mkpw.pw_set_cutoff(ctx, cfg.ecut_ry, cfg.fft)
    return (ctx,) + mkpw.pw_set_kpoints(ctx, cfg.kpts)


def test_kept_potential_leaves_room():
    # k-list, projectors and V in a budget of their own sizes, in both orders, and
    # H within it (small bases: no work array) as without a budget
    torch = torch_cuda()
    from paper_2412_01695_amd import mkpw
    rng = np.random.default_rng(3)
    c = synth.make_config(1)
    nk, n, nb = 300, 15, 4
    kpts = rng.uniform(-0.5, 0.5, (nk, 3)) @ synth.reciprocal_rows(c.lat)
    cfg = synth.Config("budget", c.lat, 13.0, (n,) * 3, kpts, nb, c.tau, c.projectors, c.dij, 9)
    v = rng.standard_normal((n,) * 3)
    res, budget = [], 0
    for order in ("bv", "vb", "free"):
        ctx, npw, npwx = _budgeted(cfg, 0 if order == "bv" else budget if order == "vb" else 0)
        try:
            beta = np.random.default_rng(4).standard_normal((nk, cfg.nproj, npwx)) + 0j
            for step in "bv" if order == "free" else order:
                if step == "b":
                    mkpw.pw_set_projectors(ctx, beta, cfg.dij)
                    if order == "bv":  # all that is held before V, and V in both precisions
                        budget = mkpw.pw_get_option(ctx, "device_bytes") + 12 * n**3
                        mkpw.pw_set_option(ctx, "hbm_budget_bytes", budget)
                else:
                    mkpw.pw_set_vloc(ctx, v)
            if order == "vb":  # the order in which something extra was kept
                assert mkpw.pw_get_option(ctx, "device_bytes") > budget
            if order != "free":
                mkpw.pw_set_option(ctx, "hbm_budget_bytes", budget + (1 << 20))
            psi = np.zeros((nk, nb, npwx), complex)
            psi[:] = np.random.default_rng(5).standard_normal(psi.shape)
            d = to_dev(torch, psi)
            out = torch.empty_like(d)
            torch.cuda.synchronize()
            mkpw.pw_h_psi(ctx, 0, nb, d, out)
            torch.cuda.synchronize()
            res.append(out.cpu().numpy())
        finally:
            mkpw.pw_destroy(ctx)
    for r in res[:2]:
        assert np.max(np.abs(r - res[2])) <= TOL64 * np.max(np.abs(res[2]))


def test_drho_in_a_box_per_k():
    # room for one box of difference bins per k and the sums over 64 chunks of k
    torch = torch_cuda()
    from paper_2412_01695_amd import mkpw
    rng = np.random.default_rng(6)
    c = synth.make_config(1)
    nk, n, nb = 100, 20, 3
    kpts = rng.uniform(-0.5, 0.5, (nk, 3)) @ synth.reciprocal_rows(c.lat)
    cfg = synth.Config("budget", c.lat, 30.0, (n,) * 3, kpts, nb, c.tau, c.projectors, c.dij, 9)
    ck, npw, npwx = _budgeted(cfg)
    cq, npwq, npwxq = _budgeted(synth.shifted(cfg, synth.q_paper()))
    try:
        mk = [mkpw.pw_get_miller(ck, ik) for ik in range(nk)]
        mq = [mkpw.pw_get_miller(cq, ik) for ik in range(nk)]
        box = np.max([(q.max(0) - k.min(0)) - (q.min(0) - k.max(0)) + 1 for k, q in zip(mk, mq)], axis=0)
        psi = rng.standard_normal((nk, nb, npwx)) + 1j * rng.standard_normal((nk, nb, npwx))
        du = rng.standard_normal((nk, nb, npwxq)) + 1j * rng.standard_normal((nk, nb, npwxq))
        d_psi, d_du = to_dev(torch, psi), to_dev(torch, du)
        outs = []
        for budget in (0, mkpw.pw_get_option(cq, "device_bytes") + 16 * nk * int(np.prod(box)) + 16 * 66 * n**3 + 20 * nk):
            mkpw.pw_set_option(cq, "hbm_budget_bytes", budget)
            out = torch.full((n,) * 3, float("nan"), dtype=torch.complex128, device="cuda")
            torch.cuda.synchronize()
            mkpw.pw_drho(cq, ck, nb, np.ones(nk) / nk, d_psi, d_du, out)
            torch.cuda.synchronize()
            outs.append(out.cpu().numpy())
        # the same sum shared out otherwise: the oracle's bound for each
        assert np.max(np.abs(outs[1] - outs[0])) <= 2e-12 * np.max(np.abs(outs[0]))
    finally:
        mkpw.pw_destroy(cq)
        mkpw.pw_destroy(ck)
