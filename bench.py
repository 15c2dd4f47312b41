"""Benchmark: batched H|psi> over many k-points on one MI355X.

    python bench.py [--gpus 1] [--steps 20] [--warmup 5] [--config 4] [--no-cpu]
                    [--no-solve] [--serve-requests N]

A step is one pw_h_psi over the whole batch of the workload (every k-point
and band in one launch, inputs resident in HBM).  The default workload is
the 1728-k-point fcc cell (ecut 40 Ry, FFT 36^3, 24 bands, 4 projectors),
the configuration of the FP64-vs-mixed metric; value is its FP64 throughput
in k-band H|psi> per second, and the same batch is timed in mixed precision
(complex64, FP32 accumulation) beside it.  The dominant kernel's roofline
fraction is computed from the flop count of the kernel that ran (the dense
product's, see `kernel_flops`, or the pruned FFT pipeline's, see
`algorithmic_work`) over its average launch time measured with HIP events on
the launch stream.  The CPU baseline is the FP64 oracle's
dense route (H_k psi_k by zgemm per k, H_k built outside the timed region),
on a process pool over the host cores.  Beside the step throughput it
reports the H|psi> throughput of the 512- and 2048-k workloads, the Davidson
time-to-solution of the headline batch (FP64 to 1e-10 and to 1e-6 Ry; mixed
precision to 1e-6 Ry, with and without its FP64 refinement; for each, the
largest eigenvalue difference over all k against the FP64 1e-10 Ry solve and
the error against the oracle's dense diagonalisation on sampled k-points,
the sample holding each solve's worst k), the
DFPT CG at q = 0 and at the paper's q, and, with --serve-requests N, the
p50/p99 latency of the continuous-batching server on a Poisson stream of N
Davidson requests (not run by default: the server process has ended twice
with a host segmentation fault during its concurrent start-up, cause not
found).  Prints one JSON line.
"""
from __future__ import annotations

import argparse
import json
import math
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_FP64_TFLOPS = 78.6    # MI355X vector FP64 (256 CU x 64 lanes x 2 x 2.4 GHz)
PEAK_FP32_TFLOPS = 157.3   # MI355X vector FP32 (packed); unpacked issue caps at 78.6
PEAK_HBM_GBS = 8000.0


# HBM bytes per launch of the H|psi> kernel from rocprofv3 counter runs
# (FETCH_SIZE, then WRITE_SIZE, KiB per dispatch), scaled by what the same
# counters read for a 1 GiB device-to-device copy (FETCH x 2.0, WRITE x 1.0),
# keyed by workload, precision and launch shape, and valid only for the kernel
# sources they were taken on (hash of the files below).
KERNEL_SOURCES = ("hpsi_dense.hip", "hpsi_dense_shape.hpp", "hpsi_types.hpp", "internal.hpp")
MEASURED_TRAFFIC = {
    ("fcc1-ecut40-fft36-1728k", "fp64", (6, 512, 0)): {
        "sources": "af43c389e8f90ac5", "fetch_kib": 347102.7, "write_kib": 331776.0,
        "fetch_scale": 2.0, "write_scale": 1.0,
        "profile": "profiles/hpsi_dense_fp64_fcc1-ecut40-fft36-1728k.md"},
    ("fcc1-ecut40-fft36-1728k", "mixed", (6, 256, 0)): {
        "sources": "af43c389e8f90ac5", "fetch_kib": 170518.0, "write_kib": 165888.0,
        "fetch_scale": 2.0, "write_scale": 1.0,
        "profile": "profiles/hpsi_dense_mixed_fcc1-ecut40-fft36-1728k.md"},
}


def progress(msg):
    """One line on stderr per finished stage (the JSON result goes to stdout)."""
    print(f"[bench {time.strftime('%H:%M:%S')}] {msg}", file=sys.stderr, flush=True)


def kernel_source_hash():
    import hashlib
    h = hashlib.sha256()
    for f in KERNEL_SOURCES:
        with open(os.path.join(ROOT, "paper_2412_01695_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def measured_traffic(workload, prec, shape):
    """Counter-measured HBM bytes per launch, or None when no counters were
    taken for this kernel source, workload and shape."""
    m = MEASURED_TRAFFIC.get((workload, prec, (shape["variant"], shape["threads"], shape["slab"])))
    if not m or m["sources"] != kernel_source_hash():
        return None
    return m["fetch_kib"] * 1024 * m["fetch_scale"] + m["write_kib"] * 1024 * m["write_scale"]


def algorithmic_work(cfg, miller_by_k, nbnd, cbytes=16, with_3pass=False):
    """Flops and I/O bytes per k-band of one H|psi>, averaged over the batch.

    Pruned FFT pair with 5 N log2 N flops per complex 1D transform of length
    N: z on the S_k occupied sticks, y on the W1_k occupied x columns of all
    N3 planes, x on all N2 N3 lines, each both ways; 2 flops per mesh point
    for V(r) u(r); 4 per plane wave for the kinetic term; 8 npw nproj for each
    of lambda = beta^H psi and beta gamma plus 8 nproj^2 for gamma = D lambda.
    I/O bytes: psi in and H psi out (cbytes per coefficient: 16 for
    complex128, 8 for complex64) plus the projector row block and the per-k
    maps (16 B per plane wave) shared by the k's bands.  With with_3pass, also
    the bytes of a three-pass (unfused) FFT that keeps the y-transformed
    planes in HBM between passes (4 W1 N^2 coefficients more per k-band): the
    bound such a design could not beat."""
    n1, n2, n3 = cfg.fft
    f1 = lambda n: 5.0 * n * math.log2(n)
    flops = 0.0
    io = 0.0
    io3 = 0.0
    for m in miller_by_k:
        npw = m.shape[0]
        s = len({(int(a), int(b)) for a, b, _ in m})
        w1 = int(m[:, 0].max() - m[:, 0].min() + 1)
        fft = 2 * (s * f1(n3) + w1 * n3 * f1(n2) + n2 * n3 * f1(n1))
        flops += fft + 2.0 * n1 * n2 * n3 + 4.0 * npw + 16.0 * npw * cfg.nproj + 8.0 * cfg.nproj ** 2
        kio = 2.0 * cbytes * npw + (cbytes * cfg.nproj * npw + 16.0 * npw) / nbnd
        io += kio
        # an unfused design keeps the W1 planes of y-transformed data in HBM
        # between its three passes: written, read and written back, read
        io3 += kio + 4.0 * w1 * n2 * n3 * cbytes
    k = len(miller_by_k)
    if with_3pass:
        return flops / k, io / k, io3 / k
    return flops / k, io / k


def _cpu_worker(cfg, ks, runs, reps, barrier, out_q):
    """One process of the CPU baseline: H_k of its k-points built (timed apart),
    then `runs` passes of H_k psi_k (zgemm) over them `reps` times, each pass
    started at the barrier shared by all processes."""
    from threadpoolctl import threadpool_limits

    from oracle import hamiltonian as ham
    from paper_2412_01695_amd import synth

    def bfn(c, ik, m):
        return synth.beta_values(c, synth.q_vectors(c, ik, m))

    with threadpool_limits(limits=1):
        t0 = time.perf_counter()
        vt = ham.vtilde(synth.vloc_grid(cfg))
        hs, ps = [], []
        for ik in ks:
            kp = ham.KPoint(cfg, int(ik), vt, bfn)
            hs.append(kp.h)
            ps.append(np.ascontiguousarray(synth.psi_guess(cfg, int(ik), kp.miller).T))
        build = time.perf_counter() - t0
        times = []
        for _ in range(runs):
            barrier.wait()
            t0 = time.perf_counter()
            for _ in range(reps):
                for h, p in zip(hs, ps):
                    h @ p
            times.append(time.perf_counter() - t0)
    out_q.put((build, times))


def cpu_baseline(cfg_ids=(4, 2, 3), k_per_core=(27, 32, 32), runs=5, reps=8):
    """The oracle's FP64 dense route, as the CPU reference of the metric: per
    k-point, H_k (npw x npw, built from the oracle's naive-DFT V~ and the
    projectors) times psi_k (npw x nbnd) in one zgemm.  One process per host
    core (BLAS single-threaded in each), a bounded sample of k-points of each
    workload split across them; H_k construction is timed separately and
    excluded; each of `runs` passes starts at a barrier and takes as long as
    its slowest process; the median pass gives k-band/s."""
    import multiprocessing as mp

    from paper_2412_01695_amd import synth
    try:
        cores = len(os.sched_getaffinity(0))
    except AttributeError:
        cores = os.cpu_count()
    ctx = mp.get_context("fork")
    res = {}
    for cid, kpc in zip(cfg_ids, k_per_core):
        cfg = synth.make_config(cid)
        nks = min(cfg.nk, kpc * cores)
        ks = np.unique(np.linspace(0, cfg.nk - 1, nks).astype(int))
        chunks = [ks[i::cores] for i in range(cores)]
        chunks = [c for c in chunks if len(c)]
        barrier = ctx.Barrier(len(chunks))
        q = ctx.Queue()
        procs = [ctx.Process(target=_cpu_worker, args=(cfg, c, runs, reps, barrier, q)) for c in chunks]
        t0 = time.perf_counter()
        for p in procs:
            p.start()
        got = [q.get() for _ in procs]
        for p in procs:
            p.join()
        wall = time.perf_counter() - t0
        per_run = np.max(np.array([g[1] for g in got]), axis=0)   # slowest process of each pass
        med = float(np.median(per_run))
        res[cfg.name] = {"value": reps * len(ks) * cfg.nbnd / med, "unit": "k-band/s", "cores": len(chunks),
                         "kind": "oracle",
                         "sample": f"{len(ks)} of {cfg.nk} k-points x {cfg.nbnd} bands, {reps} times per pass "
                                   f"(H_k psi_k zgemm, dense "
                                   f"H_k built outside the timed passes in {max(g[0] for g in got):.1f} s), "
                                   f"{len(chunks)} processes x 1 BLAS thread, median of {runs} passes "
                                   f"({med * 1e3:.1f} ms each), {wall:.1f} s wall",
                         "passes_ms": [float(x) * 1e3 for x in per_run]}
    return res


def oracle_eig_error(cfg, vloc, miller_lib, eigs, nsample=8, extra_k=()):
    """max |eig - dense eig| (Ry) on sampled k-points (evenly spaced, plus
    `extra_k`), per solve in `eigs`."""
    import scipy.linalg

    from oracle import hamiltonian as ham
    from paper_2412_01695_amd import synth

    def bfn(c, ik, m):
        return synth.beta_values(c, synth.q_vectors(c, ik, m))

    vt = ham.vtilde(vloc)
    ks = np.unique(np.concatenate([np.linspace(0, cfg.nk - 1, nsample).astype(int),
                                   np.asarray(list(extra_k), dtype=int)]))
    err = {name: 0.0 for name in eigs}
    for ik in ks:
        kp = ham.KPoint(cfg, int(ik), vt, bfn)
        if cfg.qij is None:
            ref = np.linalg.eigvalsh(kp.h)[:cfg.nbnd]
        else:
            ref = scipy.linalg.eigh(kp.h, kp.s, eigvals_only=True)[:cfg.nbnd]
        for name, e in eigs.items():
            err[name] = max(err[name], float(np.max(np.abs(e[ik] - ref))) * 2.0)
    return err, [int(k) for k in ks]


def time_davidson(torch, mkpw, sysm, prec, tol_ry):
    """Time-to-solution of one Davidson solve from the seeded guess, run twice
    from the same start: the first solve in a process also autotunes the H|psi>
    launch shape for each row count the solver applies H to (once per process,
    precision, mesh and row-count bucket) and is reported as first_seconds; the
    second is the steady state reported as seconds."""
    cfg = sysm.cfg
    guess = torch.from_numpy(sysm.psi_guess()).cuda()
    times = []
    for _ in range(2):
        psi = guess.clone()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        st, eig, iters, conv = mkpw.pw_davidson(sysm.ctx, prec, cfg.nbnd, psi, cfg.nk, tol_ry, 300)
        torch.cuda.synchronize()
        times.append(time.perf_counter() - t0)
    opt = lambda k: mkpw.pw_get_option(sysm.ctx, k)
    return {"seconds": times[1], "first_seconds": times[0], "status": int(st), "converged_k": int(conv.sum()),
            "iters_min": int(iters.min()), "iters_max": int(iters.max()), "tol_ry": tol_ry,
            "hpsi_kband_applications": opt("last_hpsi_kbands"), "iterations": opt("last_iterations"),
            "graph_replays": opt("last_graph_replays")}, eig


def dfpt_sample(torch, mkpw, cfg_id, thr=1e-24, loose_thr=1e-10):
    """Batched DFPT CG on a whole workload: occupied states from an FP64
    Davidson, rhs = -(1 - P_v) dV u with dV u taken as (T + dV) u - T u from a
    second context whose local potential is dV, then (H - eps + alpha P_v) x =
    rhs for every (k, occupied band) in one pw_dfpt_cg call, FP64 and mixed.
    The accuracy check applies A once more through pw_h_psi."""
    from paper_2412_01695_amd import synth
    from paper_2412_01695_amd.system import System

    cfg = synth.make_config(cfg_id)
    nocc = int(cfg.extra.get("nocc", cfg.nbnd))
    sysm = System(cfg, 0)
    dsys = System(cfg, 0, stream=sysm.stream, vloc=synth.dv_grid(cfg, int(cfg.extra.get("dv_seed", 7))),
                  with_projectors=False)
    torch.cuda.set_stream(sysm.stream)
    try:
        u = torch.from_numpy(sysm.psi_guess(nocc)).cuda()
        st, eig, iters, conv = mkpw.pw_davidson(sysm.ctx, mkpw.PW_FP64, nocc, u, cfg.nk, 1e-10, 300)
        # kinetic 1/2 |k+G|^2 in the library's plane-wave order, zero on the padding
        kin = np.zeros((cfg.nk, 1, sysm.npwx))
        for ik, m in enumerate(sysm.miller):
            q = synth.q_vectors(cfg, ik, m)
            kin[ik, 0, :m.shape[0]] = 0.5 * np.einsum("ij,ij->i", q, q)
        kin = torch.from_numpy(kin).cuda()
        tu = torch.empty_like(u)
        mkpw.pw_h_psi(dsys.ctx, mkpw.PW_FP64, nocc, u, tu)
        dvu = tu - kin * u
        c = torch.bmm(u.conj(), dvu.transpose(1, 2).contiguous())           # [k, mu, nu] = <u_mu|dV u_nu>
        rhs = -(dvu - torch.bmm(c.transpose(1, 2).contiguous(), u))          # -(1 - P_v) dV u
        eps = np.ascontiguousarray(eig)
        alpha = np.maximum(2.0 * (eps.max(axis=1) - eps.min(axis=1)), 0.1)
        out = {"workload": f"{cfg.name}: {cfg.nk} k, {nocc} occupied bands = rhs per k, FFT {cfg.fft[0]}^3, "
                           f"{cfg.nproj} projectors; occupied states from FP64 Davidson ({int(conv.sum())}/{cfg.nk} "
                           f"k converged)", "systems": cfg.nk * nocc, "thr": thr}
        eps_t = torch.from_numpy(eps).cuda()[:, :, None]
        a_t = torch.from_numpy(alpha).cuda()[:, None, None]
        # at the tight threshold of the parity tests, and at a looser one (|rho|
        # 1e-10, a residual norm near 1e-5) where the complex64 phase does the
        # whole solve and the FP64 phase only checks it
        runs = [("fp64", mkpw.PW_FP64, thr), ("mixed", mkpw.PW_MIXED, thr)]
        if loose_thr:
            runs += [("fp64_loose", mkpw.PW_FP64, loose_thr), ("mixed_loose", mkpw.PW_MIXED, loose_thr)]
        for name, prec, th in runs:
            times = []
            for _ in range(2):  # the first also autotunes H|psi> shapes (as in time_davidson)
                x = torch.zeros_like(rhs)
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                st, it = mkpw.pw_dfpt_cg(sysm.ctx, prec, nocc, u, eps, alpha, nocc, rhs, x, th, 2000)
                torch.cuda.synchronize()
                times.append(time.perf_counter() - t0)
            dt = times[1]
            hx = torch.empty_like(x)
            mkpw.pw_h_psi(sysm.ctx, mkpw.PW_FP64, nocc, x, hx)
            ux = torch.bmm(u.conj(), x.transpose(1, 2).contiguous())
            ax = hx - eps_t * x + a_t * torch.bmm(ux.transpose(1, 2).contiguous(), u)
            rel = (torch.linalg.vector_norm(ax - rhs, dim=2) / torch.linalg.vector_norm(rhs, dim=2)).max().item()
            out[name] = {"thr": th, "seconds": dt, "first_seconds": times[0], "status": int(st),
                         "iters_min": int(it.min()), "iters_max": int(it.max()),
                         "systems_per_s": cfg.nk * nocc / dt, "max_rel_residual": rel,
                         "hpsi_kband_applications": mkpw.pw_get_option(sysm.ctx, "last_hpsi_kbands"),
                         "graph_replays": mkpw.pw_get_option(sysm.ctx, "last_graph_replays")}
        return out
    finally:
        dsys.close()
        sysm.close()


def time_spsi(torch, mkpw, ctx, prec, nbnd, psi, spsi, steps, warmup):
    for _ in range(warmup):
        mkpw.pw_s_psi(ctx, prec, nbnd, psi, spsi)
    torch.cuda.synchronize()
    st = torch.cuda.current_stream()   # the context's stream (set by the caller)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record(st)
    for _ in range(steps):
        mkpw.pw_s_psi(ctx, prec, nbnd, psi, spsi)
    e1.record(st)
    torch.cuda.synchronize()
    return e0.elapsed_time(e1) / steps


def overlap_sample(torch, mkpw, cfg_id, steps, warmup, solve, check):
    """The workload with the model overlap S = 1 + beta q beta^H: one pw_s_psi
    over the whole batch timed like H|psi> (HBM-bound: psi in, S psi out, the
    projector rows of each k shared by its bands), and the generalized
    Davidson (H psi = eps S psi) to 1e-10 Ry in FP64 and to 1e-6 Ry mixed."""
    from paper_2412_01695_amd import synth
    from paper_2412_01695_amd.system import System

    cfg = synth.with_overlap(synth.make_config(cfg_id))
    sysm = System(cfg, 0)
    torch.cuda.set_stream(sysm.stream)
    try:
        nbnd, nkb = cfg.nbnd, cfg.nk * cfg.nbnd
        psi = torch.from_numpy(sysm.psi_guess()).cuda()
        sp = torch.empty_like(psi)
        ms = time_spsi(torch, mkpw, sysm.ctx, mkpw.PW_FP64, nbnd, psi, sp, steps, warmup)
        npw = sysm.npw.astype(np.float64)
        io = float(np.sum(2.0 * 16.0 * npw * nbnd + 16.0 * cfg.nproj * npw))
        gbs = io / (ms * 1e-3) / 1e9
        out = {"workload": f"{cfg.name}: {cfg.nk} k x {nbnd} bands, {cfg.nproj} projectors, q per atom "
                           f"s 16 / p 12 (two channels coupled 4 / 3)",
               "s_psi": {"ms_per_call": ms, "kband_per_s": nkb / (ms * 1e-3), "dtype": "c128",
                         "roofline": {"bound": "hbm", "achieved": gbs, "peak": PEAK_HBM_GBS, "unit": "GB/s",
                                      "frac": gbs / PEAK_HBM_GBS, "kernel": "spsi_mfma_kernel",
                                      "bytes_per_launch": io}}}
        eigs = {}
        for name, prec, tol in (("fp64", mkpw.PW_FP64, 1e-10), ("mixed", mkpw.PW_MIXED, 1e-6)):
            if not solve:
                break
            out[name], eigs[name] = time_davidson(torch, mkpw, sysm, prec, tol)
            out[name]["kband_per_s"] = nkb / out[name]["seconds"]
        if check and eigs:
            # the sample also holds each solve's k farthest from the FP64 solve
            worst = {int(np.abs(e - eigs["fp64"]).max(axis=1).argmax()) for e in eigs.values()}
            err, ks = oracle_eig_error(cfg, sysm.vloc, sysm.miller, eigs, extra_k=sorted(worst))
            for name in eigs:
                out[name]["max_eig_err_vs_oracle_ry"] = err[name]
            out["oracle_k_sample"] = ks
        return out
    finally:
        sysm.close()


def dfpt_q_sample(torch, mkpw, cfg_id):
    """DFPT at the paper's wavevector q on a whole workload made insulating: the
    two-atom cell with its local potential deepened until the lowest nocc bands
    are separated from the rest at every k and k+q (synth.gapped).  FP64
    Davidson at the k and k+q lists, the right-hand sides -(1 - P_v^{k+q}) dV u_k
    on the device, the CG at k+q for every (k, occupied band) in FP64 and mixed
    precision (true relative residual checked with one more H application on
    the k+q context), and the induced density of Eq. drho from the solutions."""
    from paper_2412_01695_amd import synth
    from paper_2412_01695_amd.system import System

    cfg = synth.gapped(synth.make_config(cfg_id))
    q = synth.q_paper()
    nocc = int(cfg.extra["nocc"])
    sk = System(cfg, 0)
    sq = System(synth.shifted(cfg, q), 0, stream=sk.stream)
    torch.cuda.set_stream(sk.stream)
    try:
        # the occupied bands and the first empty one (for the gap) must
        # converge; the bands above are buffer bands
        nb = int(cfg.extra.get("nb_solve", nocc + 1))
        for s in (sk, sq):
            mkpw.pw_set_option(s.ctx, "dav_nconv", nocc + 1)
        out = {"q_cart": [float(x) for x in q]}
        eig = {}
        vec = {}
        for name, s in (("k", sk), ("k+q", sq)):
            guess = torch.from_numpy(s.psi_guess(nb)).cuda()
            times = []
            for _ in range(2):  # the first also autotunes H|psi> shapes (as in time_davidson)
                u = guess.clone()
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                st, e, it, conv = mkpw.pw_davidson(s.ctx, mkpw.PW_FP64, nb, u, cfg.nk, 1e-10, 300)
                torch.cuda.synchronize()
                times.append(time.perf_counter() - t0)
            out[f"davidson_{name}_s"] = times[1]
            out[f"davidson_{name}_first_s"] = times[0]
            out[f"davidson_{name}_converged_k"] = int(conv.sum())
            eig[name], vec[name] = e, u
        ek, eq = eig["k"], eig["k+q"]
        gap = float(np.min(eq[:, nocc]) - np.max(ek[:, nocc - 1]))
        uk = vec["k"][:, :nocc].contiguous()
        uq = vec["k+q"][:, :nocc].contiguous()
        dv = synth.dv_complex_grid(cfg)
        rhs = torch.empty((cfg.nk, nocc, sq.npwx), dtype=torch.complex128, device="cuda")

        def wall(fn, reps=3):
            # the first call also grows the stream's memory pool; the rest are
            # the steady state
            ts = []
            for _ in range(reps):
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                fn()
                torch.cuda.synchronize()
                ts.append(time.perf_counter() - t0)
            return min(ts[1:]), ts[0]

        t_rhs, t_rhs_first = wall(lambda: mkpw.pw_dfpt_rhs(sq.ctx, sk.ctx, nocc, dv, uk, uq, rhs))
        npk, npq = sk.npw.astype(np.float64), sq.npw.astype(np.float64)
        pair_flops = float(np.sum(8.0 * npk * npq * nocc))
        out.update({
            "workload": f"{cfg.name} at q = (2 pi/a)(-1/8, -1/4, 3/8): {cfg.nk} k and {cfg.nk} k+q, local "
                        f"potential x{cfg.extra['vloc_scale']:g} (insulating), {nocc} occupied bands = rhs per k, "
                        f"FFT {cfg.fft[0]}^3, complex periodic dV",
            "systems": cfg.nk * nocc, "gap_kq_min_minus_k_max_ha": gap,
            "rhs_s": t_rhs, "rhs_first_s": t_rhs_first, "rhs_tflops": pair_flops / t_rhs / 1e12,
            "pair_flops": pair_flops})
        eps = np.ascontiguousarray(ek[:, :nocc])
        hi = np.maximum(ek[:, nocc - 1], eq[:, nocc - 1])
        lo = np.minimum(ek[:, 0], eq[:, 0])
        alpha = np.maximum(2.0 * (hi - lo), 0.1)
        eps_t = torch.from_numpy(eps).cuda()[:, :, None]
        a_t = torch.from_numpy(alpha).cuda()[:, None, None]
        x = None
        for name, prec in (("cg_fp64", mkpw.PW_FP64), ("cg_mixed", mkpw.PW_MIXED)):
            times = []
            for _ in range(2):
                x = torch.zeros_like(rhs)
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                st, it = mkpw.pw_dfpt_cg(sq.ctx, prec, nocc, uq, eps, alpha, nocc, rhs, x, 1e-24, 2000)
                torch.cuda.synchronize()
                times.append(time.perf_counter() - t0)
            hx = torch.empty_like(x)
            mkpw.pw_h_psi(sq.ctx, mkpw.PW_FP64, nocc, x, hx)
            ux = torch.bmm(uq.conj(), x.transpose(1, 2).contiguous())
            ax = hx - eps_t * x + a_t * torch.bmm(ux.transpose(1, 2).contiguous(), uq)
            rel = (torch.linalg.vector_norm(ax - rhs, dim=2) / torch.linalg.vector_norm(rhs, dim=2)).max().item()
            out[name] = {"seconds": times[1], "first_seconds": times[0], "status": int(st),
                         "iters_min": int(it.min()), "iters_max": int(it.max()),
                         "systems_per_s": cfg.nk * nocc / times[1], "max_rel_residual": rel,
                         "hpsi_kband_applications": mkpw.pw_get_option(sq.ctx, "last_hpsi_kbands")}
        w = np.full(cfg.nk, 1.0 / cfg.nk)
        drho = torch.empty(cfg.fft, dtype=torch.complex128, device="cuda")
        t_rho, t_rho_first = wall(lambda: mkpw.pw_drho(sq.ctx, sk.ctx, nocc, w, uk, x, drho))
        out.update({"drho_s": t_rho, "drho_first_s": t_rho_first, "drho_tflops": pair_flops / t_rho / 1e12})
        return out
    finally:
        sq.close()
        sk.close()


def serving_sample(n, rate=20.0, timeout_s=900):
    """The serving stream in a server process of its own (the serve module's
    entry point): the measurement is that of a server that has done nothing
    else, and a failure there is reported here instead of ending this run."""
    import subprocess
    cmd = [sys.executable, "-u", "-m", "paper_2412_01695_amd.serve", "--requests", str(n), "--rate", str(rate)]
    try:
        p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=None, cwd=os.path.dirname(os.path.abspath(__file__)),
                           timeout=timeout_s, text=True)
    except subprocess.TimeoutExpired:
        return {"error": f"server process did not finish within {timeout_s} s", "command": " ".join(cmd[1:])}
    except OSError as e:
        return {"error": f"server process could not be started: {e}", "command": " ".join(cmd[1:])}
    lines = [x for x in p.stdout.splitlines() if x.startswith("{")]
    if p.returncode != 0 or not lines:
        how = f"signal {-p.returncode}" if p.returncode < 0 else f"exit code {p.returncode}"
        return {"error": f"server process ended with {how}", "command": " ".join(cmd[1:])}
    return json.loads(lines[-1])


def kernel_flops(variant, cfg, npw, flops_kb):
    """(kernel, flops per k-band) of the kernel that ran: variant 6 is the dense
    product (8 npw^2 for the local term, 16 npw nproj for the projectors),
    otherwise the pruned transforms' count `flops_kb`."""
    if variant != 6:
        return "hpsi_kernel", flops_kb
    n = np.asarray(npw, float)
    return "hpsi_dense_kernel", float(np.mean(8.0 * n * n + 16.0 * n * cfg.nproj))


def hpsi_sample(torch, mkpw, cid, steps, warmup):
    """FP64 and mixed H|psi> throughput of another whole workload, with the
    roofline fractions of its autotuned kernels."""
    from paper_2412_01695_amd import synth
    from paper_2412_01695_amd.system import System

    cfg = synth.make_config(cid)
    s = System(cfg, 0)
    torch.cuda.set_stream(s.stream)
    try:
        psi64 = torch.from_numpy(s.psi_guess()).cuda()
        h64 = torch.empty_like(psi64)
        psi32 = psi64.to(torch.complex64)
        h32 = torch.empty_like(psi32)
        nkb = cfg.nk * cfg.nbnd
        flops_kb, io_kb = algorithmic_work(cfg, s.miller, cfg.nbnd, 16)
        out = {"config": f"{cfg.nk} k-points (npw {int(s.npw.min())}-{int(s.npw.max())}), {cfg.nbnd} bands, "
                         f"FFT {cfg.fft[0]}^3, {cfg.nproj} projectors", "flops_per_kband": flops_kb}
        for name, prec, psi, h, peak in (("fp64", mkpw.PW_FP64, psi64, h64, PEAK_FP64_TFLOPS),
                                         ("mixed", mkpw.PW_MIXED, psi32, h32, PEAK_FP32_TFLOPS)):
            ms, _ = time_hpsi(torch, mkpw, s.ctx, prec, cfg.nbnd, psi, h, steps, warmup)
            kern, kern_flops = kernel_flops(mkpw.pw_get_option(s.ctx, "hpsi_variant_tuned"), cfg, s.npw, flops_kb)
            tf = kern_flops * nkb / (ms * 1e-3) / 1e12
            out[name] = {"ms_per_call": ms, "kband_per_s": nkb / (ms * 1e-3), "tflops": tf, "roofline_frac": tf / peak,
                         "kernel": kern, "kernel_flops_per_kband": kern_flops,
                         "shape": {k: mkpw.pw_get_option(s.ctx, f"hpsi_{k}_tuned")
                                   for k in ("variant", "slab", "threads")}}
        return cfg.name, out
    finally:
        s.close()


def time_hpsi(torch, mkpw, ctx, prec, nbnd, psi, hpsi, steps, warmup):
    for _ in range(warmup):
        mkpw.pw_h_psi(ctx, prec, nbnd, psi, hpsi)
    torch.cuda.synchronize()
    st = torch.cuda.current_stream()   # the context's stream (set by the caller)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    t0 = time.perf_counter()
    e0.record(st)
    for _ in range(steps):
        mkpw.pw_h_psi(ctx, prec, nbnd, psi, hpsi)
    e1.record(st)
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    return e0.elapsed_time(e1) / steps, wall * 1e3 / steps


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--config", type=int, default=4)
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--no-solve", action="store_true")
    # the serving stream is off by default: its server process has ended twice
    # with a host segmentation fault during the concurrent start-up of its
    # first 48 requests on 8 slots, and the cause is not found
    ap.add_argument("--serve-requests", type=int, default=0)
    ap.add_argument("--other-configs", default="2,3",
                    help="workloads whose H|psi> throughput is reported beside the headline ('' to skip)")
    ap.add_argument("--dfpt-config", type=int, default=3, help="workload of the DFPT CG sample (0: skip)")
    ap.add_argument("--overlap-config", type=int, default=2,
                    help="workload of the overlap (S psi, generalized Davidson) sample (0: skip)")
    ap.add_argument("--only", choices=["fp64", "mixed", "both"], default="both")
    ap.add_argument("--shape", default=None,
                    help="fix the H|psi> launch shape as variant,threads,slab (e.g. 1,256,10) instead of "
                         "autotuning, for profiles that must time one known kernel")
    ap.add_argument("--tune-log", action="store_true", help="print the autotuner's candidate timings to stderr")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="after the timed steps, run one 1 GiB device-to-device copy (a known-size "
                         "reference dispatch for HBM byte counters)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(json.dumps({"error": "this library runs on one GPU; the k-point list shards across GPUs "
                                   "as independent pools, which this benchmark does not launch",
                          "n_gpus": args.gpus}))
        sys.exit(2)

    import torch
    from paper_2412_01695_amd import mkpw, synth
    from paper_2412_01695_amd.system import System

    cfg = synth.make_config(args.config)
    torch.cuda.set_device(0)
    sysm = System(cfg, 0)
    torch.cuda.set_stream(sysm.stream)
    nbnd = cfg.nbnd
    psi_h = sysm.psi_guess()
    psi64 = torch.from_numpy(psi_h).cuda()
    h64 = torch.empty_like(psi64)
    psi32 = psi64.to(torch.complex64)
    h32 = torch.empty_like(psi32)
    nkb = cfg.nk * nbnd
    flops_kb, io64_kb, io64_3p = algorithmic_work(cfg, sysm.miller, nbnd, 16, True)
    _, io32_kb, io32_3p = algorithmic_work(cfg, sysm.miller, nbnd, 8, True)

    if args.tune_log:
        mkpw.pw_set_option(sysm.ctx, "tune_log", 1)
    if args.shape:
        sv = [int(x) for x in args.shape.split(",")]
        mkpw.pw_set_option(sysm.ctx, "hpsi_variant", sv[0])
        mkpw.pw_set_option(sysm.ctx, "hpsi_threads", sv[1])
        mkpw.pw_set_option(sysm.ctx, "hpsi_slab", sv[2])

    def shape():
        return {k: mkpw.pw_get_option(sysm.ctx, f"hpsi_{k}_tuned") for k in ("variant", "slab", "threads")}

    out, shapes = {}, {}
    if args.only in ("fp64", "both"):
        ms64, wall64 = time_hpsi(torch, mkpw, sysm.ctx, mkpw.PW_FP64, nbnd, psi64, h64, args.steps, args.warmup)
        out["fp64"], shapes["fp64"] = ms64, shape()
        progress(f"H|psi> fp64 {cfg.name}: {ms64:.4f} ms")
    if args.only in ("mixed", "both"):
        ms32, wall32 = time_hpsi(torch, mkpw, sysm.ctx, mkpw.PW_MIXED, nbnd, psi32, h32, args.steps, args.warmup)
        out["mixed"], shapes["mixed"] = ms32, shape()
        progress(f"H|psi> mixed {cfg.name}: {ms32:.4f} ms")

    if args.copy_calibration:
        a = torch.empty(1 << 27, dtype=torch.float64, device="cuda")
        b = torch.empty_like(a)
        a.fill_(1.0)
        torch.cuda.synchronize()
        b.copy_(a)
        torch.cuda.synchronize()
        del a, b

    key = "fp64" if "fp64" in out else "mixed"
    ms = out[key]
    io_kb = io64_kb if key == "fp64" else io32_kb
    io_3p = io64_3p if key == "fp64" else io32_3p
    value = nkb / (ms * 1e-3)
    kern, kern_flops = kernel_flops(shapes[key]["variant"], cfg, sysm.npw, flops_kb)
    flops_launch = kern_flops * nkb
    achieved_tf = flops_launch / (ms * 1e-3) / 1e12
    res = {
        "metric": "k-band H|psi>/s (FP64 vs mixed FP32) at 1e-6 Ry; p50/p99 solve latency",
        "value": value,
        "unit": "k-band/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "c128" if key == "fp64" else "c64",
        "data": "synthetic",
        "config": {"workload": f"{cfg.name}: fcc a=7.6 bohr, {len(cfg.tau)} atom(s), ecut {cfg.ecut_ry:g} Ry, "
                               f"FFT {cfg.fft[0]}^3, {cfg.nk} k-points (npw {int(sysm.npw.min())}-"
                               f"{int(sysm.npw.max())}), {nbnd} bands, {cfg.nproj} projectors; one pw_h_psi "
                               f"over all {nkb} k-band rows per step",
                   "global_batch": nkb, "parallelism": "single GPU, all k in one launch"},
        "roofline": {"bound": "alu", "achieved": achieved_tf,
                     "peak": PEAK_FP64_TFLOPS if key == "fp64" else PEAK_FP32_TFLOPS,
                     "unit": "TFLOP/s",
                     "frac": achieved_tf / (PEAK_FP64_TFLOPS if key == "fp64" else PEAK_FP32_TFLOPS),
                     "traffic": measured_traffic(cfg.name, key, shapes[key]),
                     "traffic_unit": "HBM bytes per launch (counters; null if not taken on this kernel)",
                     "kernel": kern, "shape": shapes[key], "flops_per_kband": kern_flops,
                     "io_bytes_per_launch": io_kb * nkb,
                     "hbm_io_GBs": io_kb * nkb / (ms * 1e-3) / 1e9,
                     "hbm_frac": io_kb * nkb / (ms * 1e-3) / 1e9 / PEAK_HBM_GBS,
                     "hbm_3pass_bound_kband_s": PEAK_HBM_GBS * 1e9 / io_3p,
                     "vs_hbm_3pass_bound": value / (PEAK_HBM_GBS * 1e9 / io_3p)},
    }
    if "mixed" in out and "fp64" in out:
        res["mixed"] = {"value": nkb / (out["mixed"] * 1e-3), "ms_per_step": out["mixed"], "dtype": "c64",
                        "shape": shapes["mixed"],
                        "speedup_vs_fp64": out["fp64"] / out["mixed"],
                        "roofline_frac": kernel_flops(shapes["mixed"]["variant"], cfg, sysm.npw, flops_kb)[1]
                        * nkb / (out["mixed"] * 1e-3) / 1e12 / PEAK_FP32_TFLOPS,
                        "traffic": measured_traffic(cfg.name, "mixed", shapes["mixed"]),
                        "io_bytes_per_launch": io32_kb * nkb}
    eigs = {}
    if not args.no_solve:
        solve = {}
        # FP64 to 1e-10 Ry (the parity tolerance) and to the metric's 1e-6 Ry,
        # mixed to 1e-6 Ry with and without its FP64 refinement
        # (the last: complex64 only, its phase ending at residual 2e-5, not 2e-4)
        for name, prec, tol, refine, rt in (("fp64", mkpw.PW_FP64, 1e-10, 1, 2000),
                                            ("fp64_1e-6", mkpw.PW_FP64, 1e-6, 1, 2000),
                                            ("mixed", mkpw.PW_MIXED, 1e-6, 1, 2000),
                                            ("mixed_before_refinement", mkpw.PW_MIXED, 1e-6, 0, 2000),
                                            ("mixed_before_refinement_rtol2e-5", mkpw.PW_MIXED, 1e-6, 0, 200)):
            mkpw.pw_set_option(sysm.ctx, "mixed_refine", refine)
            mkpw.pw_set_option(sysm.ctx, "mixed_switch_rtol_e7", rt)
            solve[name], eigs[name] = time_davidson(torch, mkpw, sysm, prec, tol)
            solve[name]["kband_per_s"] = nkb / solve[name]["seconds"]
            progress(f"Davidson {name}: {solve[name]['seconds']:.4f} s")
        mkpw.pw_set_option(sysm.ctx, "mixed_refine", 1)
        mkpw.pw_set_option(sysm.ctx, "mixed_switch_rtol_e7", 2000)
        # every k, every band: eigenvalues against the FP64 solve to 1e-10 Ry
        # (itself checked against the oracle on a k sample below)
        for name in eigs:
            solve[name]["max_eig_diff_vs_fp64_1e-10_all_k_ry"] = float(2.0 * np.abs(eigs[name] - eigs["fp64"]).max())
        progress("max |eig - FP64 1e-10| over all k (Ry): " +
                 ", ".join(f"{n} {solve[n]['max_eig_diff_vs_fp64_1e-10_all_k_ry']:.2e}" for n in eigs))
        res["solve"] = solve
    if not args.no_cpu:
        if eigs:
            # the sample also holds each solve's k farthest from the FP64 solve
            worst = {int(np.abs(e - eigs["fp64"]).max(axis=1).argmax()) for e in eigs.values()}
            err, ks = oracle_eig_error(cfg, sysm.vloc, sysm.miller, eigs, extra_k=sorted(worst))
            for name in eigs:
                res["solve"][name]["max_eig_err_vs_oracle_ry"] = err[name]
            res["solve"]["oracle_k_sample"] = ks
            progress(f"oracle eigenvalue errors (Ry): {err}")
    sysm.close()
    if args.other_configs:
        res["hpsi_workloads"] = {}
        for cid in (int(x) for x in args.other_configs.split(",")):
            if cid != args.config:
                name, entry = hpsi_sample(torch, mkpw, cid, args.steps, args.warmup)
                res["hpsi_workloads"][name] = entry
                progress(f"H|psi> {name}: fp64 {entry['fp64']['ms_per_call']:.4f} ms, "
                         f"mixed {entry['mixed']['ms_per_call']:.4f} ms")
    if not args.no_cpu:
        allcpu = cpu_baseline()
        progress("cpu baseline: " + ", ".join(f"{k} {v['value']:.0f} k-band/s" for k, v in allcpu.items()))
        res["cpu_baseline"] = dict(allcpu.get(cfg.name) or next(iter(allcpu.values())))
        res["cpu_baseline_workloads"] = allcpu
    if args.overlap_config > 0:
        res["overlap"] = overlap_sample(torch, mkpw, args.overlap_config, args.steps, args.warmup,
                                        not args.no_solve, not args.no_cpu)
        progress("overlap sample done")
    if args.dfpt_config > 0:
        res["dfpt"] = dfpt_sample(torch, mkpw, args.dfpt_config)
        progress("DFPT q = 0 done")
        res["dfpt_q"] = dfpt_q_sample(torch, mkpw, args.dfpt_config)
        progress("DFPT q != 0 done")
    if args.serve_requests <= 0:
        res["serving"] = {"skipped": "not run by default: the server process ended twice with a host "
                                     "segmentation fault during the concurrent start-up of its first 48 "
                                     "requests on 8 slots; cause not found (--serve-requests N runs it)"}
    else:
        res["serving"] = serving_sample(args.serve_requests)
        if "error" in res["serving"]:
            progress(f"serving: {res['serving']['error']}")
        else:
            progress(f"serving: p50 {res['serving']['p50_s']:.3f} s, p99 {res['serving']['p99_s']:.3f} s")
    print(json.dumps(res))


if __name__ == "__main__":
    main()
