#!/usr/bin/env python
"""Benchmark: auxiliary-Kalman MCMC steps/s on one MI355X.

Workload: the d_x = 64, T = 4096 latent field on a periodic grid (nearest-
neighbour F, squared-exponential Q + 1e-6 jitter) observed through Student-t
noise (nu = 3, scale 0.5) at 32 evenly spaced sites; second-order proposal,
fixed step size delta; one chain.  Synthetic data and normals, all seeded.

One "step" is one full auxiliary-Kalman MH step: aux draw + linearisation,
parallel filter (block fold, tree, block re-scan), pathwise sampler (element
build, fold, tree, final), reverse linearisation + filter, MH reduction and
select.  Inputs (model, data, normals, uniforms) are resident in HBM before
the timed region starts.

Prints ONE JSON line (rank 0).  With --gpus > 1 it exits with a message: this
build measures a single GPU.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

import numpy as np

METRIC = "aux-Kalman MCMC steps/s at d_x=64,T=4096; batched+adjoint vs plain, same GPU"
PEAK_FP64_TFLOPS = 78.6  # MI355X dense FP64 (vector and matrix)
PEAK_HBM_GBS = 8000.0


def fold_flops_per_step(d: int, first: bool, t0: bool) -> float:
    """Algorithmic flops of one block-fold step at dimension d (2 per multiply-
    add, triangular and symmetric products counted at their reduced cost):
    predict F C F' (2 GEMMs), Cholesky + triangular inverse of S, X = L^{-1} P^p,
    X'X, and for blocks past the first F A, Y = L^{-1} F A, Y'Y, X'Y."""
    d3 = float(d) ** 3
    f = (0.0 if t0 else 4.0 * d3) + (2.0 / 3.0) * d3 + 2.0 * d3
    if not first:
        f += 2.0 * d3 + d3 + d3 + 2.0 * d3
    return f


def fold_flops_per_launch(N: int, d: int, B: int) -> float:
    tot = 0.0
    for t in range(N):
        tot += fold_flops_per_step(d, first=(t < B), t0=(t == 0))
    return tot


TRAFFIC_FILE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "profiles",
                            "filter_fold_latent_field_traffic.txt")
KERNEL_SOURCES = ("paper_2303_00301_amd/csrc/akf_team.hpp",
                  "paper_2303_00301_amd/csrc/akf_internal.h",
                  "paper_2303_00301_amd/csrc/akf_kernels.hip")


FIXED_TRAFFIC_FILE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "profiles",
                                  "first_order_mfold_latent_field_traffic.txt")
FIXED_SOURCES = ("paper_2303_00301_amd/csrc/akf_team.hpp",
                 "paper_2303_00301_amd/csrc/akf_internal.h",
                 "paper_2303_00301_amd/csrc/akf_fixed.hip")


def timed_launches(lib, _lib, family: str, capacity: int, fn):
    """Run fn() with HIP-event timing on every launch of one kernel family;
    returns (average launch ms, launches) or (None, 0)."""
    import ctypes as C
    _lib.check(lib.akf_timing_enable(_lib.FAMILIES[family], capacity), "akf_timing_enable")
    fn()
    n_l, k_ms = C.c_int32(), C.c_double()
    _lib.check(lib.akf_timing_collect(C.byref(n_l), C.byref(k_ms)), "akf_timing_collect")
    lib.akf_timing_enable(-1, 0)
    return (k_ms.value / n_l.value, n_l.value) if n_l.value else (None, 0)


def roofline_obj(bound: str, kernel: str, work: float, avg_ms, peak: float, unit: str,
                 scale: float, traffic=None) -> dict:
    """work per launch (flops or bytes) / average launch time, against peak."""
    if avg_ms is None:
        return None
    achieved = work / (avg_ms * 1e-3) / scale
    return {"bound": bound, "kernel": kernel, "achieved": achieved, "peak": peak, "unit": unit,
            "frac": achieved / peak, "traffic": traffic, "avg_launch_ms": avg_ms,
            "work_per_launch": work}


def _digest(sources) -> str:
    import hashlib
    h = hashlib.sha256()
    root = os.path.dirname(os.path.abspath(__file__))
    for rel in sources:
        with open(os.path.join(root, rel), "rb") as f:
            h.update(f.read())
    return h.hexdigest()


def kernel_source_digest() -> str:
    return _digest(KERNEL_SOURCES)


def fixed_source_digest() -> str:
    return _digest(FIXED_SOURCES)


def _traffic(path: str, digest: str, block: int):
    try:
        with open(path) as f:
            kv = dict(line.split(":", 1) for line in f if ":" in line and not line.startswith("#"))
    except OSError:
        return None
    kv = {k.strip(): v.strip() for k, v in kv.items()}
    if kv.get("kernel_source_sha256") != digest:
        return None
    if int(kv.get("scan_block", "-1")) != block:
        return None
    return float(kv["traffic_bytes_per_launch"])


def measured_traffic(block: int):
    """HBM bytes per fold launch from the committed FETCH_SIZE / WRITE_SIZE
    counter summary, or None when there is none, it was taken at another scan
    block size, or the kernel sources changed since it was taken."""
    return _traffic(TRAFFIC_FILE, kernel_source_digest(), block)


def measured_fixed_traffic(block: int):
    """The same for k_mfold<64> of the first-order run."""
    return _traffic(FIXED_TRAFFIC_FILE, fixed_source_digest(), block)


def auto_block(N: int, d: int) -> int:
    D = 16 if d <= 16 else (32 if d <= 32 else 64)
    teams = 1 if D == 64 else (4 if D == 32 else 8)
    target = 256 * teams
    B = max(2 if D > 16 and N <= 512 else 4, (N + target - 1) // target)
    return min(B, N)


def host_info() -> dict:
    """The host the oracle runs on: CPU model and the number of logical CPUs."""
    model = "unknown"
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    return {"cpu_model": model, "nproc": os.cpu_count()}


def oracle_threads() -> int:
    """Host threads for the oracle's multi-chain baselines: every core of the
    GPU's share of the host (at most 16)."""
    return max(1, min(16, os.cpu_count() or 1))


def adj_build_flops_per_step(d: int, p: int) -> float:
    """Algorithmic flops of one step of the adjoint element build (2 per
    multiply-add): the predicted moments F P^f F' + Q (4 d^3), H P^p and
    S = H P^p H' + R (2 p d^2 + 2 p^2 d), S^{-1} (p^3), K = (H P^p)' S^{-1},
    Sig H, H' Sig H, F K and (F K) H."""
    return 4.0 * d ** 3 + 8.0 * p * d * d + 6.0 * p * p * d + p ** 3


def adj_grad_flops_per_step(d: int, p: int) -> float:
    """Algorithmic flops of one step of the adjoint's gradient contractions:
    the same recomputed filter quantities as the element build, K, Pbar F,
    (Pbar F) P^f, F' Pbar F, S^{-1} H P^p, K' Fbar and (K' Fbar) P^f."""
    return 10.0 * d ** 3 + 6.0 * p * d * d + 6.0 * p * p * d + p ** 3


def cpu_baseline(w, n_steps: int, order=None, delta=None) -> dict:
    """The FP64 oracle (sequential C, one thread) on a bounded sample: n_steps
    full MH steps of the same workload, from the same state and normals."""
    import numpy as np
    import oracle
    order = w.order if order is None else order
    delta = w.delta if delta is None else delta
    M = oracle.Model(**w.oracle_kwargs())
    xi = w.normals(n_steps)
    un = w.uniforms(n_steps)
    x = w.x_true.copy()
    t0 = time.perf_counter()
    for k in range(n_steps):
        r = oracle.mh_step(M, w.y, x, delta, order, xi[k, 0], xi[k, 1], un[k])
        x = r["x_out"]
    dt = time.perf_counter() - t0
    return {"value": n_steps / dt, "unit": "steps/s", "cores": 1, "kind": "oracle",
            "sample": f"{n_steps} full MH steps of order {order} on the same workload "
                      f"(d_x={w.dx}, T={w.N}) by the sequential FP64 C oracle on one host "
                      f"thread (one chain is a sequential computation), {dt:.1f} s",
            "seconds": dt, **host_info()}


def bench_batched(torch, S, W, _lib, K: int, dev, cpu: bool = False) -> dict:
    """512 ragged chains (N ~ U{128..8192}, d ~ U{4,16,32}, Poisson log link):
    K steps as one batched plan (hipGraph replay) vs 512 sequential plain runs
    of the same K steps from the same start, same normals, same scan blocks;
    their results are compared chain by chain.  Rooflines of the batched
    filter fold and sampler element build per team width, from an eager run
    with event timing."""
    import ctypes as C
    import tempfile
    lib = _lib.load()
    t0 = time.perf_counter()
    ws = W.ragged_poisson_batch()
    gen = torch.Generator(device=dev)
    gen.manual_seed(104)
    chains = []
    for w in ws:
        y = torch.as_tensor(w.y, dtype=torch.float64, device=dev)
        x0 = torch.log(y + 0.5).contiguous()
        chains.append(dict(model=S.DeviceModel.from_workload(w, device=dev), y=y, x=x0.clone(),
                           x0=x0, delta=w.delta, order=2,
                           xi=torch.randn((K, 2, w.N, w.dx), dtype=torch.float64, device=dev,
                                          generator=gen),
                           unif=torch.rand((K,), dtype=torch.float64, device=dev,
                                           generator=gen).clamp_(min=1e-300),
                           accepted=torch.empty(K, dtype=torch.int32, device=dev),
                           log_ratio=torch.empty(K, dtype=torch.float64, device=dev),
                           status=torch.empty(K, dtype=torch.int32, device=dev)))
    t_setup = time.perf_counter() - t0
    cache = os.path.join(tempfile.gettempdir(), "auxkf_batch_tune.jsonl")
    t0 = time.perf_counter()
    plan = S.BatchPlan(chains, K, block=0, tune_cache=cache, device=dev)
    torch.cuda.synchronize()
    t_plan = time.perf_counter() - t0
    info = plan.info()
    blk = {c["D"]: c["block"] for c in info["classes"]}
    plan.run(use_graph=True)  # warm-up: captures the graph
    torch.cuda.synchronize()
    # per-class rooflines from an eager run (events around each launch), then
    # the timed graph replays from the start state
    roof = {}
    fams = [(f"kb_fold<{D}>", f"batch_fold{D}", D, "fold") for D in sorted(blk)]
    fams += [(f"kb_sbuild<{D}>", f"batch_sbuild{D}", D, "sbuild") for D in sorted(blk)]
    for kname, fam, D, kind in fams:
        for c in chains:
            c["x"].copy_(c["x0"])
        torch.cuda.synchronize()
        _lib.check(lib.akf_timing_enable(_lib.FAMILIES[fam], 4 * K + 8), "akf_timing_enable")
        plan.run(use_graph=False)
        n_l, k_ms = C.c_int32(), C.c_double()
        _lib.check(lib.akf_timing_collect(C.byref(n_l), C.byref(k_ms)), "akf_timing_collect")
        lib.akf_timing_enable(-1, 0)
        if not n_l.value:
            continue
        mine = [w for w in ws if (16 if w.dx <= 16 else 32 if w.dx <= 32 else 64) == D]
        if kind == "fold":
            work = sum(fold_flops_per_launch(w.N, w.dx, blk[D]) for w in mine)
        else:
            work = sum(8.0 * w.dx ** 3 * w.N for w in mine)
        roof[kname] = roofline_obj("mfma", kname, work, k_ms.value / n_l.value,
                                   PEAK_FP64_TFLOPS, "TFLOP/s", 1e12)
        roof[kname]["launches"] = n_l.value
        if D == 16:  # the timed phase also runs the d <= 4 chains, one lane per item
            lane = "kl_phase<0> (fold)" if kind == "fold" else "kl_phase<2> (sampler build)"
            roof[kname]["includes"] = lane + " for the d <= 4 chains, one lane per item"
    for c in chains:
        c["x"].copy_(c["x0"])
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record(plan.stream)
    plan.run(use_graph=True)
    e1.record(plan.stream)
    torch.cuda.synchronize()
    ms_batched = e0.elapsed_time(e1)
    acc = float(torch.stack([c["accepted"].float().mean() for c in chains]).mean().item())
    # plain per-chain launches, same inputs, start and blocks
    wsp = S.Workspace(dev)
    blk_of = lambda c: blk[16 if c["model"].dx <= 16 else 32]
    xs = [c["x0"].clone() for c in chains]
    for c, x in zip(chains, xs):  # warm-up (workspace growth, code load)
        S.mh_run(c["model"], c["y"], x, c["delta"], 2, c["xi"][:1], c["unif"][:1],
                 block=blk_of(c), ws=wsp, outputs=False)
    xs = [c["x0"].clone() for c in chains]
    outs = []
    torch.cuda.synchronize()
    e0.record()
    for c, x in zip(chains, xs):
        outs.append(S.mh_run(c["model"], c["y"], x, c["delta"], 2, c["xi"], c["unif"],
                             block=blk_of(c), ws=wsp))
    e1.record()
    torch.cuda.synchronize()
    ms_plain = e0.elapsed_time(e1)
    # chain-by-chain agreement of the two runs
    max_dx, max_dlr, n_dec, n_status = 0.0, 0.0, 0, 0
    for w, c, x, o in zip(ws, chains, xs, outs):
        n_status += int((c["status"] != o["status"]).sum().item())
        same = bool(torch.equal(c["accepted"], o["accepted"]))
        n_dec += 0 if same else 1
        ok = (o["status"] == 0)
        if bool(ok.any()):
            d_lr = (c["log_ratio"] - o["log_ratio"]).abs()[ok]
            max_dlr = max(max_dlr, float(d_lr.max().item()))
        if same:
            err = float(torch.linalg.norm(c["x"] - x).item()) / max(
                1.0, float(torch.linalg.norm(x).item()))
            max_dx = max(max_dx, err)
    n_ch = len(chains)
    plan.close()
    out = {"workload": "512 chains, N ~ U{128..8192}, d_x ~ U{4,16,32}, random stable F, "
                       "Q = 0.1 I, Poisson log link, order 2",
           "steps": K, "chains": n_ch, "time_steps": int(sum(w.N for w in ws)),
           "batched_ms_per_step": ms_batched / K, "plain_ms_per_step": ms_plain / K,
           "batched_chain_steps_per_s": n_ch * K / (ms_batched * 1e-3),
           "plain_chain_steps_per_s": n_ch * K / (ms_plain * 1e-3),
           "speedup_vs_plain": ms_plain / ms_batched,
           "batched_time_steps_per_s": sum(w.N for w in ws) * K / (ms_batched * 1e-3),
           "acceptance": acc, "classes": info["classes"], "plan_s": t_plan,
           "setup_s": t_setup,
           "equality_vs_plain": {
               "same_start_and_normals": True,
               "max_rel_path_diff": max_dx,
               "max_abs_log_ratio_diff": max_dlr,
               "chains_with_a_different_decision": n_dec,
               "status_mismatches": n_status},
           "roofline": roof}
    if cpu:
        out["cpu_baseline"] = batched_cpu_baseline(ws)
    return out


def batched_cpu_baseline(ws, n_chains: int = 64) -> dict:
    """The oracle steps the first n_chains chains once each, one chain per host
    thread (the C oracle releases the interpreter lock), on every core of the
    GPU's share of the host; its rate in time steps per second is comparable
    with batched_time_steps_per_s."""
    import numpy as np
    import oracle
    from concurrent.futures import ThreadPoolExecutor
    sample = ws[:n_chains]
    oracle.lib()

    def one(w):
        xi = w.normals(1)[0]
        oracle.mh_step(oracle.Model(**w.oracle_kwargs()), w.y, np.log(w.y + 0.5), w.delta, 2,
                       xi[0], xi[1], float(w.uniforms(1)[0]))

    nt = oracle_threads()
    t0 = time.perf_counter()
    with ThreadPoolExecutor(max_workers=nt) as ex:
        list(ex.map(one, sample))
    dt = time.perf_counter() - t0
    n_ts = sum(w.N for w in sample)
    return {"value": n_ts / dt, "unit": "time steps/s", "cores": nt, "kind": "oracle",
            "sample": f"one MH step of each of the first {len(sample)} chains ({n_ts} time "
                      f"steps) by the sequential FP64 C oracle, one chain per thread on "
                      f"{nt} host threads, {dt:.1f} s",
            **host_info()}


def bench_adjoint(torch, S, W, _lib, reps: int, dev, cpu: bool = False) -> dict:
    """log p(y | theta) and its reverse-mode adjoint, d_x = 32, d_y = 16, T = 16384;
    rooflines of the adjoint's two matrix kernels (per-step gradient
    contractions, element build)."""
    lib = _lib.load()
    pw = W.lgssm_params()
    model = S.LGSSM(pw.m0, pw.P0, pw.y, device=dev)
    th = [torch.as_tensor(a, dtype=torch.float64, device=dev).contiguous()
          for a in (pw.theta0.F, pw.theta0.logq, pw.theta0.H, pw.theta0.logr)]
    ws = S.Workspace(dev)
    S.lgssm_loglik(model, *th, ws=ws)
    S.lgssm_loglik_grad(model, *th, ws)
    torch.cuda.synchronize()
    e = [torch.cuda.Event(enable_timing=True) for _ in range(3)]
    tf, tb = [], []
    for _ in range(reps):
        e[0].record()
        S.lgssm_loglik(model, *th, ws=ws)
        e[1].record()
        S.lgssm_loglik_grad(model, *th, ws)
        e[2].record()
        torch.cuda.synchronize()
        tf.append(e[0].elapsed_time(e[1]))
        tb.append(e[1].elapsed_time(e[2]))
    tf.sort()
    tb.sort()
    mf, mb = tf[len(tf) // 2], tb[len(tb) // 2]
    N, d, p = pw.N, pw.m0.shape[0], pw.y.shape[1]
    roof = {}
    for fam, kname, per_step in (("adj_grad", "k_adj_grad<32>", adj_grad_flops_per_step(d, p)),
                                 ("adj_build", "k_adj_build<32>",
                                  adj_build_flops_per_step(d, p))):
        def run():
            for _ in range(reps):
                S.lgssm_loglik(model, *th, ws=ws)
                S.lgssm_loglik_grad(model, *th, ws)
            torch.cuda.synchronize()

        avg, n_l = timed_launches(lib, _lib, fam, 2 * reps + 4, run)
        roof[kname] = roofline_obj("mfma", kname, per_step * N, avg, PEAK_FP64_TFLOPS,
                                   "TFLOP/s", 1e12)
        if roof[kname] is not None:
            roof[kname]["launches"] = n_l
    out = {"workload": "LGSSM d_x=32, d_y=16, T=16384, theta = (F, log diag Q, H, log diag R), "
                       "1584 parameters",
           "forward_ms": mf, "adjoint_ms": mb,
           "adjoint_time_steps_per_s": pw.N / ((mf + mb) * 1e-3),
           "adjoint_over_forward": mb / mf,
           "roofline": roof}
    if cpu:
        # the oracle's log-likelihood and its gradient (the Fisher score, from the
        # smoother) on the same series
        import oracle
        t = pw.theta0
        t0 = time.perf_counter()
        oracle.lgssm_loglik(pw.m0, pw.P0, t.F, t.logq, t.H, t.logr, pw.y)
        oracle.fisher_score(pw.m0, pw.P0, t.F, t.logq, t.H, t.logr, pw.y)
        dt = time.perf_counter() - t0
        out["cpu_baseline"] = {"value": pw.N / dt, "unit": "time steps/s", "cores": 1,
                               "kind": "oracle",
                               "sample": f"log-likelihood and gradient over the same {pw.N} "
                                         f"steps by the sequential FP64 C oracle on one host "
                                         f"thread (a sequential computation), {dt:.1f} s",
                               **host_info()}
    return out


def bench_gibbs(torch, S, W, _lib, n_sweeps: int, dev, cpu: bool = False) -> dict:
    """Gibbs sweeps over (theta, x) at the differentiation workload's shape
    (d_x = 32, d_y = 16, T = 16384, 1584 parameters): MALA on theta with the
    log-likelihood and adjoint at each proposal, an exact refresh of x and one
    auxiliary Kalman path step per sweep, all on the device.  The normals are
    drawn on the device beforehand (a seeded torch generator), outside the
    timed region.  The adjoint's share is the time of one log-likelihood +
    gradient evaluation (timed alone on the same theta) over the sweep time."""
    pw = W.lgssm_params()
    N, dx, dy = pw.N, pw.m0.shape[0], pw.y.shape[1]
    p = S.n_theta(dx, dy)
    sd, eps, k = 10.0, 2e-4, 1
    model = S.LGSSM(pw.m0, pw.P0, pw.y, device=dev)
    theta0 = torch.as_tensor(pw.theta0.flat(), dtype=torch.float64, device=dev)
    x0 = torch.zeros((N, dx), dtype=torch.float64, device=dev)
    gen = torch.Generator(device=dev)
    gen.manual_seed(105)

    def draws(n):
        return (torch.randn((n, p), generator=gen, dtype=torch.float64, device=dev),
                torch.rand((n, 1), generator=gen, dtype=torch.float64, device=dev),
                torch.randn((n, N, dx), generator=gen, dtype=torch.float64, device=dev),
                torch.randn((n, k, 2, N, dx), generator=gen, dtype=torch.float64, device=dev),
                torch.rand((n, k), generator=gen, dtype=torch.float64, device=dev))

    G = S.gibbs_init(model, theta0, x0, prior_sd=sd)
    warm = draws(3)
    for i in range(3):
        S.gibbs_sweep(G, eps, warm[0][i], warm[1][i], warm[2][i], 0.5, warm[3][i], warm[4][i],
                      outputs=False)
    dr = draws(n_sweeps)
    acc_t = torch.zeros(n_sweeps, dtype=torch.int32, device=dev)
    acc_p = torch.zeros(n_sweeps, dtype=torch.int32, device=dev)
    outs = []
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for i in range(n_sweeps):
        outs.append(S.gibbs_sweep(G, eps, dr[0][i], dr[1][i], dr[2][i], 0.5, dr[3][i], dr[4][i]))
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / n_sweeps
    for i, o in enumerate(outs):
        acc_t[i] = o["accepted_theta"][0]
        acc_p[i] = o["path_accepted"][0]
    # one log-likelihood + gradient evaluation on the same shape
    F, lq, H, lr = (t.contiguous() for t in (G.theta[:dx * dx].view(dx, dx),
                                              G.theta[dx * dx:dx * dx + dx],
                                              G.theta[dx * dx + dx:dx * dx + dx + dy * dx]
                                              .view(dy, dx),
                                              G.theta[dx * dx + dx + dy * dx:]))
    ws = S.Workspace(dev)
    S.lgssm_loglik(model, F, lq, H, lr, ws=ws)
    S.lgssm_loglik_grad(model, F, lq, H, lr, ws)
    torch.cuda.synchronize()
    e0.record()
    for _ in range(5):
        S.lgssm_loglik(model, F, lq, H, lr, ws=ws)
        S.lgssm_loglik_grad(model, F, lq, H, lr, ws)
    e1.record()
    torch.cuda.synchronize()
    ll_ms = e0.elapsed_time(e1) / 5
    out = {"workload": f"Gibbs sweeps over (theta, x), LGSSM d_x={dx}, d_y={dy}, T={N}, "
                       f"{p} parameters, prior N(0, {sd:g}^2), MALA step {eps:g}, {k} path step "
                       f"per sweep",
           "sweeps": n_sweeps, "ms_per_sweep": ms, "sweeps_per_s": 1e3 / ms,
           "time_steps_per_s": N * 1e3 / ms,
           "theta_acceptance": float(acc_t.float().mean().item()),
           "path_acceptance": float(acc_p.float().mean().item()),
           "loglik_and_adjoint_ms": ll_ms, "adjoint_share": ll_ms / ms,
           "final_status": [int(v) for v in G.status.cpu().tolist()]}
    if cpu:
        import numpy as np
        from oracle import gibbs as OG
        rng = np.random.default_rng(105)
        th = pw.theta0.flat()
        t0 = time.perf_counter()
        lp, g = OG.gibbs_init(pw.m0, pw.P0, pw.y, th, sd)
        t1 = time.perf_counter()
        OG.gibbs_sweep(pw.m0, pw.P0, pw.y, th, lp, g, np.zeros((N, dx)), sd, eps,
                       rng.standard_normal(p), 0.5, rng.standard_normal((N, dx)), 0.5,
                       rng.standard_normal((k, 2, N, dx)), np.array([0.5]))
        dt = time.perf_counter() - t1
        out["cpu_baseline"] = {"value": 1.0 / dt, "unit": "sweeps/s", "cores": 1,
                               "kind": "oracle",
                               "sample": f"one sweep of the same shape by the oracle (FP64 C "
                                         f"Kalman filter, Fisher-identity score, RTS sampler "
                                         f"and MH step on one host thread), {dt:.1f} s "
                                         f"(plus {t1 - t0:.1f} s for its starting gradient)",
                               **host_info()}
    return out


def bench_stoch_vol(torch, S, W, _lib, K: int, dev, cpu_steps: int = 0) -> dict:
    """Second paper workload on the same path: multivariate stochastic volatility
    (d_x = 30, T = 250), one chain, both linearisation orders; roofline of the
    filter fold (32-wide teams), the oracle timed beside it."""
    lib = _lib.load()
    out = {"workload": "stoch_vol_d30_T250: F = 0.9 I, equicorrelated Q (tau 2, rho 0.25), "
                       "y ~ N(0, exp(x)) per coordinate, one chain"}
    for order in (1, 2):
        w = W.stoch_vol(order=order)
        M = S.DeviceModel.from_workload(w, device=dev)
        y = torch.as_tensor(w.y, dtype=torch.float64, device=dev)
        x = torch.as_tensor(w.x_true, dtype=torch.float64, device=dev).contiguous()
        gen = torch.Generator(device=dev)
        gen.manual_seed(60 + order)
        xi = torch.randn((K + 2, 2, w.N, w.dx), dtype=torch.float64, device=dev, generator=gen)
        un = torch.rand((K + 2,), dtype=torch.float64, device=dev, generator=gen).clamp_(min=1e-300)
        ws = S.Workspace(dev)
        S.mh_run(M, y, x, w.delta, order, xi[:2], un[:2], ws=ws)
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        box = {}

        def run():
            e0.record()
            box["r"] = S.mh_run(M, y, x, w.delta, order, xi[2:], un[2:], ws=ws)
            e1.record()
            torch.cuda.synchronize()

        avg, _ = timed_launches(lib, _lib, "filter_fold", 4 * K + 8, run)
        r = box["r"]
        ms = e0.elapsed_time(e1) / K
        B = auto_block(w.N, w.dx)
        res = {"delta": w.delta, "ms_per_step": ms, "steps_per_s": 1000.0 / ms,
               "acceptance": r["accepted"].float().mean().item(),
               "roofline": roofline_obj("mfma", "k_filter_fold<32>",
                                        fold_flops_per_launch(w.N, w.dx, B), avg,
                                        PEAK_FP64_TFLOPS, "TFLOP/s", 1e12)}
        if cpu_steps > 0:
            progress("cpu_baseline ...")
            res["cpu_baseline"] = cpu_baseline(w, cpu_steps, order=order)
        out[f"order{order}"] = res
    return out


def bench_obs_linearisation(torch, S, W, _lib, K: int, dev, cpu_steps: int = 0) -> dict:
    """Order 3 on the quadratic-observation field (d_x = 64, T = 4096, 32 sites,
    y = z + 0.2 z^2 + N(0, 0.25)): the proposal takes the Gaussian fitted to the
    observation model around the path in place of log h's own derivatives.
    One chain; the linearisation changes only the elementwise kernels, so the
    step costs what the Student-t field's order-2 step costs.  Roofline of the
    filter fold; the oracle's order-3 step timed beside it."""
    lib = _lib.load()
    w = W.quadratic_obs_field()
    M = S.DeviceModel.from_workload(w, device=dev)
    y = torch.as_tensor(w.y, dtype=torch.float64, device=dev).contiguous()
    x = torch.as_tensor(w.x_true, dtype=torch.float64, device=dev).contiguous()
    gen = torch.Generator(device=dev)
    gen.manual_seed(109)
    xi = torch.randn((K + 2, 2, w.N, w.dx), dtype=torch.float64, device=dev, generator=gen)
    un = torch.rand((K + 2,), dtype=torch.float64, device=dev, generator=gen).clamp_(min=1e-300)
    ws = S.Workspace(dev)
    S.mh_run(M, y, x, w.delta, 3, xi[:2], un[:2], ws=ws)
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    box = {}

    def run():
        e0.record()
        box["r"] = S.mh_run(M, y, x, w.delta, 3, xi[2:], un[2:], ws=ws)
        e1.record()
        torch.cuda.synchronize()

    avg, _ = timed_launches(lib, _lib, "filter_fold", 4 * K + 8, run)
    r = box["r"]
    ms = e0.elapsed_time(e1) / K
    B = auto_block(w.N, w.dx)
    res = {"workload": f"quadratic_obs_field_d{w.dx}_T{w.N}: latent-field dynamics, "
                       f"y = z + {w.obs_beta} z^2 + N(0, {w.scale}^2) at 32 sites, order 3 "
                       f"(reference variance {w.slr_var}), one chain",
           "delta": w.delta, "steps": K, "ms_per_step": ms, "steps_per_s": 1000.0 / ms,
           "time_steps_per_s": 1000.0 / ms * w.N,
           "acceptance": r["accepted"].float().mean().item(),
           "rejected_by_status": int((r["status"] != 0).sum().item()),
           "roofline": roofline_obj("mfma", "k_filter_fold<64>",
                                    fold_flops_per_launch(w.N, w.dx, B), avg,
                                    PEAK_FP64_TFLOPS, "TFLOP/s", 1e12)}
    if cpu_steps > 0:
        progress("cpu_baseline ...")
        res["cpu_baseline"] = cpu_baseline(w, cpu_steps, order=3)
    return res


def bench_poisson(torch, S, W, _lib, K: int, dev, cpu_steps: int = 0) -> dict:
    """Poisson AR(1) workload (d_x = 8, T = 1024, delta 0.2, order 2, one chain):
    at this size one step moves well under a megabyte and runs a few dozen
    dependent launches, so it is bound by launch and scan-level latency.
    Reported: ms per step, and per kernel family the launches per step and
    microseconds per step (each family timed with events in a run of its
    own; the families cover every launch of the step)."""
    lib = _lib.load()
    w = W.poisson_ar1()
    M = S.DeviceModel.from_workload(w, device=dev)
    y = torch.as_tensor(w.y, dtype=torch.float64, device=dev)
    x = torch.log(y + 0.5).contiguous()
    gen = torch.Generator(device=dev)
    gen.manual_seed(62)
    xi = torch.randn((K + 2, 2, w.N, w.dx), dtype=torch.float64, device=dev, generator=gen)
    un = torch.rand((K + 2,), dtype=torch.float64, device=dev, generator=gen).clamp_(min=1e-300)
    ws = S.Workspace(dev)
    S.mh_run(M, y, x, w.delta, 2, xi[:2], un[:2], ws=ws)
    torch.cuda.synchronize()
    x0 = x.clone()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    r = S.mh_run(M, y, x, w.delta, 2, xi[2:], un[2:], ws=ws)
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / K
    phases = {}
    for fam in ("lin", "filter_fold", "filter_up", "filter_final", "samp_build", "samp_fold",
                "samp_up", "samp_down", "samp_final", "mh"):
        x.copy_(x0)
        box = {}

        def run():
            S.mh_run(M, y, x, w.delta, 2, xi[2:], un[2:], ws=ws)
            torch.cuda.synchronize()

        avg, n_l = timed_launches(lib, _lib, fam, 64 * K + 8, run)
        if n_l:
            phases[fam] = {"launches_per_step": n_l / K, "us_per_step": 1000.0 * avg * n_l / K}
    out = {"workload": f"poisson_ar1_d{w.dx}_T{w.N}: F = 0.95 I, Q = 0.2 I, Poisson log link "
                       f"at every coordinate, delta {w.delta}, order 2, one chain",
           "ms_per_step": ms, "steps_per_s": 1000.0 / ms,
           "time_steps_per_s": w.N * 1000.0 / ms,
           "acceptance": r["accepted"].float().mean().item(),
           "launches_per_step": sum(p["launches_per_step"] for p in phases.values()),
           "phases": phases}
    if cpu_steps > 0:
        out["cpu_baseline"] = cpu_baseline_from(w, np.log(w.y + 0.5), cpu_steps, 2, w.delta)
    return out


def cpu_baseline_from(w, x0, n_steps: int, order: int, delta: float) -> dict:
    """The oracle's MH steps of one chain from x0 on one host thread."""
    import oracle
    M = oracle.Model(**w.oracle_kwargs())
    xi = w.normals(n_steps)
    un = w.uniforms(n_steps)
    x = x0.copy()
    t0 = time.perf_counter()
    for k in range(n_steps):
        x = oracle.mh_step(M, w.y, x, delta, order, xi[k, 0], xi[k, 1], un[k])["x_out"]
    dt = time.perf_counter() - t0
    return {"value": n_steps / dt, "unit": "steps/s", "cores": 1, "kind": "oracle",
            "sample": f"{n_steps} MH steps of order {order} on the same workload by the "
                      f"sequential FP64 C oracle on one host thread, {dt:.1f} s",
            **host_info()}


def bench_first_order(torch, S, W, _lib, K: int, dev, cpu_steps: int = 0) -> dict:
    """First-order steps on the latent-field workload (d_x = 64, T = 4096): the
    plain step, which forms the auxiliary model's covariances every step, and
    the run that forms them once per call (the first step pays for it).  The
    roofline is that of the filtering-mean block fold (k_mfold<64>): per
    launch it reads every kept S_t^{-1} (T d^2 doubles), omega and log det S
    and writes one vector per block."""
    import ctypes as C
    lib = _lib.load()
    w = W.latent_field()
    delta = 0.2 * w.delta
    M = S.DeviceModel.from_workload(w, device=dev)
    y = torch.as_tensor(w.y, dtype=torch.float64, device=dev)
    gen = torch.Generator(device=dev)
    gen.manual_seed(71)
    xi = torch.randn((K + 2, 2, w.N, w.dx), dtype=torch.float64, device=dev, generator=gen)
    un = torch.rand((K + 2,), dtype=torch.float64, device=dev, generator=gen).clamp_(min=1e-300)
    out = {"workload": f"latent_field_d{w.dx}_T{w.N}, order-1 proposal, delta {delta:.3g}, "
                       f"one chain, {K} steps per call"}
    for key, reuse in (("plain", False), ("matrices_once_per_call", True)):
        ws = S.Workspace(dev)
        x = torch.as_tensor(w.x_true, dtype=torch.float64, device=dev).contiguous()
        S.mh_run(M, y, x, delta, 1, xi[:2], un[:2], ws=ws, reuse_matrices=reuse)
        torch.cuda.synchronize()
        if reuse:
            _lib.check(lib.akf_timing_enable(_lib.FAMILIES["fixed_mean_fold"], 2 * K + 8),
                       "akf_timing_enable")
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        r = S.mh_run(M, y, x, delta, 1, xi[2:], un[2:], ws=ws, reuse_matrices=reuse)
        e1.record()
        torch.cuda.synchronize()
        ms = e0.elapsed_time(e1) / K
        out[key] = {"ms_per_step": ms, "steps_per_s": 1000.0 / ms,
                    "acceptance": r["accepted"].float().mean().item(),
                    "rejected_by_status": int((r["status"] != 0).sum().item())}
        if reuse:
            n_l, k_ms = C.c_int32(), C.c_double()
            _lib.check(lib.akf_timing_collect(C.byref(n_l), C.byref(k_ms)), "akf_timing_collect")
            lib.akf_timing_enable(-1, 0)
            if n_l.value > 0:
                N, d, D = w.N, w.dx, 64
                nb = -(-N // auto_block(N, d))
                nbytes = 8.0 * (N * D * D + N * d + N + nb * D)
                avg_ms = k_ms.value / n_l.value
                gbs = nbytes / (avg_ms * 1e-3) / 1e9
                out[key]["roofline"] = {"bound": "hbm", "kernel": "k_mfold<64>",
                                        "achieved": gbs, "peak": PEAK_HBM_GBS, "unit": "GB/s",
                                        "frac": gbs / PEAK_HBM_GBS,
                                        "traffic": measured_fixed_traffic(auto_block(N, d)),
                                        "avg_launch_ms": avg_ms, "launches": n_l.value,
                                        "bytes_per_launch": nbytes}
    out["speedup"] = out["plain"]["ms_per_step"] / out["matrices_once_per_call"]["ms_per_step"]
    if cpu_steps > 0:
        out["cpu_baseline"] = cpu_baseline(w, cpu_steps, order=1, delta=delta)
    return out


def bench_reuse(torch, S, W, _lib, K: int, dev) -> dict:
    """The headline workload (latent field, d_x = 64, T = 4096, order 2) run
    plainly and with the matrices of a forward proposal reused by the next one
    after a rejection (akf_mh_run_reuse, which decides each step's branch on
    the device and issues the launches of both, gated).  Both runs take the
    same normals and uniforms from the same state, so they make the same
    decisions.  The roofline is that of the filter fold, which every step's
    reverse proposal (and every full forward one) runs; its launches are timed
    in the plain run, since the reuse run's gated-off fold launches (which exit
    at once) would enter the same average."""
    import ctypes as C
    lib = _lib.load()
    w = W.latent_field()
    M = S.DeviceModel.from_workload(w, device=dev)
    y = torch.as_tensor(w.y, dtype=torch.float64, device=dev)
    gen = torch.Generator(device=dev)
    gen.manual_seed(97)
    xi = torch.randn((K + 2, 2, w.N, w.dx), dtype=torch.float64, device=dev, generator=gen)
    un = torch.rand((K + 2,), dtype=torch.float64, device=dev, generator=gen).clamp_(min=1e-300)
    out = {"workload": f"latent_field_d{w.dx}_T{w.N}, order-2 proposal, delta {w.delta}, "
                       f"one chain, {K} steps per call"}
    for key, reuse in (("plain", False), ("reuse_after_reject", True)):
        ws = S.Workspace(dev)
        x = torch.as_tensor(w.x_true, dtype=torch.float64, device=dev).contiguous()
        S.mh_run(M, y, x, w.delta, 2, xi[:2], un[:2], ws=ws, reuse_matrices=reuse)
        torch.cuda.synchronize()
        if not reuse:
            _lib.check(lib.akf_timing_enable(_lib.FAMILIES["filter_fold"], 4 * K + 8),
                       "akf_timing_enable")
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        r = S.mh_run(M, y, x, w.delta, 2, xi[2:], un[2:], ws=ws, reuse_matrices=reuse)
        e1.record()
        torch.cuda.synchronize()
        ms = e0.elapsed_time(e1) / K
        out[key] = {"ms_per_step": ms, "steps_per_s": 1000.0 / ms,
                    "acceptance": r["accepted"].float().mean().item(),
                    "rejected_by_status": int((r["status"] != 0).sum().item())}
        if not reuse:
            n_l, k_ms = C.c_int32(), C.c_double()
            _lib.check(lib.akf_timing_collect(C.byref(n_l), C.byref(k_ms)), "akf_timing_collect")
            lib.akf_timing_enable(-1, 0)
            if n_l.value > 0:
                B = auto_block(w.N, w.dx)
                avg_ms = k_ms.value / n_l.value
                achieved = fold_flops_per_launch(w.N, w.dx, B) / (avg_ms * 1e-3) / 1e12
                out[key]["roofline"] = {"bound": "mfma", "kernel": "k_filter_fold<64>",
                                        "achieved": achieved, "peak": PEAK_FP64_TFLOPS,
                                        "unit": "TFLOP/s", "frac": achieved / PEAK_FP64_TFLOPS,
                                        "traffic": measured_traffic(B),
                                        "avg_launch_ms": avg_ms, "launches": n_l.value}
    out["speedup"] = out["plain"]["ms_per_step"] / out["reuse_after_reject"]["ms_per_step"]
    return out


def bench_spatio_temporal(torch, S, W, _lib, K: int, dev, cpu_steps: int) -> dict:
    """Second paper workload: the spatio-temporal model (8 x 8 lattice, T = 1024,
    multivariate-t observations with nu = 1), first order, one chain.  The
    factorised step (64 scalar filters/samplers) is the product path; the dense
    step on the same model is timed beside it."""
    import ctypes as C
    w = W.spatio_temporal()
    Md = S.DeviceModel.from_workload(w, device=dev)
    Mf = Md.diagonal()
    y = torch.as_tensor(w.y, dtype=torch.float64, device=dev)
    gen = torch.Generator(device=dev)
    gen.manual_seed(80)
    xi = torch.randn((K + 3, 2, w.N, w.dx), dtype=torch.float64, device=dev, generator=gen)
    un = torch.rand((K + 3,), dtype=torch.float64, device=dev, generator=gen).clamp_(min=1e-300)
    out = {"workload": "spatio_temporal_8x8_T1024: random walks (sigma_x = 1) on an 8 x 8 "
                       "lattice, multivariate-t observations (nu = 1, precision tau^D, tau = -1/4, "
                       "D <= 1), first-order proposal, one chain",
           "delta": w.delta}
    lib = _lib.load()
    for name, M, fact, k in (("factorised", Mf, True, K), ("dense", Md, False, max(2, K // 10))):
        x = torch.as_tensor(w.x_true, dtype=torch.float64, device=dev).contiguous()
        ws = S.Workspace(dev)
        S.mh_run(M, y, x, w.delta, 1, xi[:3], un[:3], ws=ws, factorised=fact)
        torch.cuda.synchronize()
        if fact:
            _lib.check(lib.akf_timing_enable(_lib.FAMILIES["fact_scan"], 2 * k + 8),
                       "akf_timing_enable")
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        r = S.mh_run(M, y, x, w.delta, 1, xi[3:3 + k], un[3:3 + k], ws=ws, factorised=fact)
        e1.record()
        torch.cuda.synchronize()
        ms = e0.elapsed_time(e1) / k
        res = {"ms_per_step": ms, "steps_per_s": 1000.0 / ms,
               "acceptance": r["accepted"].float().mean().item(), "steps": k}
        if fact:
            n_l, k_ms = C.c_int32(), C.c_double()
            _lib.check(lib.akf_timing_collect(C.byref(n_l), C.byref(k_ms)), "akf_timing_collect")
            lib.akf_timing_enable(-1, 0)
            if n_l.value:
                avg = k_ms.value / n_l.value
                res["k_fact_scan_avg_us"] = 1000.0 * avg
                # about 60 scalar FP64 operations per (time step, coordinate) for the
                # filter and the sampler together, a division or square root as one
                res["roofline"] = roofline_obj("alu", "k_fact_scan", 60.0 * w.N * w.dx, avg,
                                               PEAK_FP64_TFLOPS, "TFLOP/s", 1e12)
        out[name] = res
    out["paper_reference"] = ("0.52 ms per iteration for the parallel-in-time auxiliary Kalman "
                              "sampler on an RTX 3090 (another machine: context only)")
    if cpu_steps > 0:
        import oracle
        Mo = oracle.Model(**w.oracle_kwargs())
        xin = w.normals(cpu_steps)
        uin = w.uniforms(cpu_steps)
        xc = w.x_true.copy()
        t0 = time.perf_counter()
        for k in range(cpu_steps):
            rr = oracle.mh_step_factorised(Mo, w.y, xc, w.delta, 1, xin[k, 0], xin[k, 1], uin[k])
            xc = rr["x_out"]
        dt = time.perf_counter() - t0
        out["cpu_baseline"] = {"value": cpu_steps / dt, "unit": "steps/s", "cores": 1,
                               "kind": "oracle",
                               "sample": f"{cpu_steps} factorised MH steps of the same workload by "
                                         f"the sequential FP64 C oracle on one host thread, "
                                         f"{dt:.1f} s", **host_info()}
    return out


def bench_lorenz(torch, S, W, _lib, K: int, dev, cpu_steps: int) -> dict:
    """Nonlinear dynamics: the Lorenz-63 SDE of the paper's diffusion-smoothing
    experiment (N = 10001 fine steps, d = 3, sparse Gaussian observations) and a
    Lorenz-96 ring (d = 40, N = 2048, Student-t observations), one chain each,
    second order, extended linearisation at x and x* every step."""
    lib = _lib.load()
    out = {}
    for name, w in (("lorenz63", W.lorenz63()), ("lorenz96", W.lorenz96())):
        M = S.DeviceModel.from_workload(w, device=dev)
        y = torch.as_tensor(w.y, dtype=torch.float64, device=dev)
        x = torch.as_tensor(w.x_true, dtype=torch.float64, device=dev).contiguous()
        gen = torch.Generator(device=dev)
        gen.manual_seed(90)
        xi = torch.randn((K + 2, 2, w.N, w.dx), dtype=torch.float64, device=dev, generator=gen)
        un = torch.rand((K + 2,), dtype=torch.float64, device=dev, generator=gen).clamp_(min=1e-300)
        ws = S.Workspace(dev)
        S.mh_run(M, y, x, w.delta, w.order, xi[:2], un[:2], ws=ws)
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        box = {}

        def run():
            e0.record()
            box["r"] = S.mh_run(M, y, x, w.delta, w.order, xi[2:], un[2:], ws=ws)
            e1.record()
            torch.cuda.synchronize()

        avg, _ = timed_launches(lib, _lib, "filter_fold", 4 * K + 8, run)
        r = box["r"]
        ms = e0.elapsed_time(e1) / K
        D = 16 if w.dx <= 16 else (32 if w.dx <= 32 else 64)
        res = {"workload": w.name, "d_x": w.dx, "T": w.N, "delta": w.delta, "ms_per_step": ms,
               "steps_per_s": 1000.0 / ms, "acceptance": r["accepted"].float().mean().item(),
               "roofline": roofline_obj("mfma", f"k_filter_fold<{D}>",
                                        fold_flops_per_launch(w.N, w.dx, auto_block(w.N, w.dx)),
                                        avg, PEAK_FP64_TFLOPS, "TFLOP/s", 1e12)}
        if cpu_steps > 0:
            import oracle
            Mo = oracle.Model(**w.oracle_kwargs())
            xin = w.normals(cpu_steps)
            uin = w.uniforms(cpu_steps)
            xc = w.x_true.copy()
            t0 = time.perf_counter()
            for k in range(cpu_steps):
                rr = oracle.mh_step(Mo, w.y, xc, w.delta, w.order, xin[k, 0], xin[k, 1], uin[k])
                xc = rr["x_out"]
            dt = time.perf_counter() - t0
            res["cpu_baseline"] = {"value": cpu_steps / dt, "unit": "steps/s", "cores": 1,
                                   "kind": "oracle",
                                   "sample": f"{cpu_steps} MH steps of the same workload by the "
                                             f"sequential FP64 C oracle on one host thread, "
                                             f"{dt:.1f} s", **host_info()}
        out[name] = res
    out["paper_reference"] = ("Lorenz-63 run of 2,500 adaptation + 1e5 steps (with a parameter "
                              "Gibbs step) in 3,149 s on an RTX 3090, about 31 ms per iteration "
                              "(another machine: context only)")
    return out


def bench_samplers(torch, S, W, _lib, K: int, dev, cpu: bool = False) -> dict:
    """The two pathwise samplers on the same filtering moments (latent field,
    d = 64, T = 4096, pseudo-observations x + N(0, delta/2)): the prefix-sum
    sampler of the MH step (element build + suffix scan) and the
    divide-and-conquer sampler (bisection tree of bridges).  Rooflines: the
    prefix-sum sampler's element build (8 d^3 per step) and the whole
    divide-and-conquer sampler (8 d^3 per leaf step, 14 d^3 per midpoint)."""
    lib = _lib.load()
    w = W.latent_field()
    M = S.DeviceModel.from_workload(w, device=dev)
    gen = torch.Generator(device=dev)
    gen.manual_seed(70)
    x = torch.as_tensor(w.x_true, dtype=torch.float64, device=dev)
    om = (x + (0.5 * w.delta) ** 0.5 * torch.randn(x.shape, dtype=torch.float64, device=dev,
                                                   generator=gen)).contiguous()
    Om = torch.full_like(om, 0.5 * w.delta)
    mf, Pf, _, _ = S.aux_filter(M, om, Om)
    xi = torch.randn((K + 1, w.N, w.dx), dtype=torch.float64, device=dev, generator=gen)
    out = {"workload": f"filtering moments of latent_field_d{w.dx}_T{w.N}"}
    d, N = w.dx, w.N
    work = {"prefix_sum": ("samp_build", "k_samp_build<64>", 8.0 * d ** 3 * N),
            "divide_and_conquer": ("dnc", "the divide-and-conquer sampler (all its launches)",
                                   8.0 * d ** 3 * N + 14.0 * d ** 3 * (N - 2))}
    for name, fn in (("prefix_sum", S.rts_sample), ("divide_and_conquer", S.dnc_sample)):
        ws = S.Workspace(dev)
        fn(M, mf, Pf, xi[0], ws=ws)
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)

        def run():
            e0.record()
            for k in range(K):
                fn(M, mf, Pf, xi[k + 1], ws=ws)
            e1.record()
            torch.cuda.synchronize()

        fam, kname, flops = work[name]
        avg, _ = timed_launches(lib, _lib, fam, 2 * K + 8, run)
        out[name + "_ms"] = e0.elapsed_time(e1) / K
        out[name + "_roofline"] = roofline_obj("mfma", kname, flops, avg, PEAK_FP64_TFLOPS,
                                               "TFLOP/s", 1e12)
    if cpu:
        out["cpu_baseline"] = sampler_cpu_baseline(w, mf, Pf)
    return out


def bench_sqrt(torch, S, W, _lib, K: int, dev, cpu: bool = False) -> dict:
    """Square-root filter and sampler (akf_sqrt_filter_sample) in FP32 and FP64
    beside the covariance-form FP64 filter and sampler (akf_aux_filter +
    akf_rts_sample) on the same pseudo-observations, with each one's largest
    error against the oracle: relative on filtering means and covariances,
    absolute per step on the log-likelihood, in smoothing sd on the path.
    Workloads: the stochastic-volatility auxiliary model (d = 30, T = 250, the
    paper's FP32 case) and a d = 32, T = 4096 model with cond(Q) = 1e6 and
    pseudo-observation variances 0.01-0.05."""
    import time
    import numpy as np
    import oracle

    def errs(res, ref, x_ref, sd):
        mf, Pf = res["mf"], res["Pf"]
        sc = np.maximum(np.linalg.norm(ref["mf"], axis=1), np.sqrt(np.einsum("tii->t", ref["Pf"])))
        return {"mean_rel": float((np.linalg.norm(mf - ref["mf"], axis=1) / sc).max()),
                "cov_rel": float((np.linalg.norm(Pf - ref["Pf"], axis=(1, 2)) /
                                  np.linalg.norm(ref["Pf"], axis=(1, 2))).max()),
                "ell_abs": float(np.abs(res["ell"] - ref["ell"]).max()),
                "path_sd": float((np.abs(res["x"] - x_ref) / sd).max())}

    cases = {}
    w = W.stoch_vol(order=2)
    rng = np.random.default_rng(6)
    u = w.x_true + np.sqrt(w.delta / 2) * rng.standard_normal(w.x_true.shape)
    om, Om, _, _ = oracle.linearise(oracle.Model(**w.oracle_kwargs()), w.y, w.x_true, u,
                                    w.delta, 2)
    Om = np.stack([np.diag(o) for o in Om]) if Om.ndim == 3 else Om
    cases["stoch_vol_d30_T250"] = (w.m0, w.P0, w.F, w.b, w.Q, om, Om)
    rng = np.random.default_rng(32)
    d, N = 32, 4096
    G = rng.standard_normal((d, d))
    F = 0.9 * G / np.max(np.abs(np.linalg.eigvals(G)))
    Uo, _ = np.linalg.qr(rng.standard_normal((d, d)))
    Q = (Uo * (np.logspace(0, -6, d) * 0.1)) @ Uo.T
    Q = 0.5 * (Q + Q.T)
    cases["cond1e6_d32_T4096"] = (np.zeros(d), np.eye(d), F, None, Q,
                                  0.5 * rng.standard_normal((N, d)),
                                  rng.uniform(0.01, 0.05, (N, d)))
    out = {}
    for name, (m0, P0, F, b, Q, om, Om) in cases.items():
        N, d = om.shape
        xi = np.random.default_rng(7).standard_normal((N, d))
        t0 = time.perf_counter()
        ref = oracle.kf(m0, P0, F, Q, np.eye(d), np.stack([np.diag(o) for o in Om]), om, b=b,
                        R_per_t=True)
        x_ref, _ = oracle.rts_sample(F, ref["mf"], ref["Pf"], ref["mp"], ref["Pp"], xi)
        t_or = time.perf_counter() - t0
        _, Ps, _, _ = oracle.rts_smooth(F, ref["mf"], ref["Pf"], ref["mp"], ref["Pp"])
        sd = np.sqrt(np.einsum("tii->ti", Ps))
        M = S.DeviceModel.from_arrays(N, m0, P0, F, Q, W.EMIT_POISSON_LOG, b=b, device=dev)
        T_ = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device=dev)
        om_d, Om_d, xi_d = T_(om), T_(Om), T_(xi)
        res = {"N": N, "d": d}

        def time_it(fn):
            fn()
            torch.cuda.synchronize()
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(K):
                r = fn()
            e1.record()
            torch.cuda.synchronize()
            return e0.elapsed_time(e1) / K, r

        for dt in ("f32", "f64"):
            ws = S.Workspace(dev)
            ms, r = time_it(lambda: S.sqrt_filter_sample(M, om_d, Om_d, xi_d, dtype=dt, ws=ws))
            Uf = r["Uf"].cpu().numpy()
            got = {"mf": r["mf"].cpu().numpy(), "Pf": Uf @ np.transpose(Uf, (0, 2, 1)),
                   "ell": r["ell"].cpu().numpy(), "x": r["x"].cpu().numpy()}
            res[f"sqrt_{dt}"] = {"ms": ms, "status": int(r["status"].item()),
                                 "error_vs_oracle": errs(got, ref, x_ref, sd)}
        ws = S.Workspace(dev)

        def cov_form():
            mf, Pf, ell, st = S.aux_filter(M, om_d, Om_d, ws=ws)
            x, st2 = S.rts_sample(M, mf, Pf, xi_d, ws=ws)
            return dict(mf=mf, Pf=Pf, ell=ell, x=x, status=st)

        ms, r = time_it(cov_form)
        got = {k: r[k].cpu().numpy() for k in ("mf", "Pf", "ell", "x")}
        res["covariance_f64"] = {"ms": ms, "status": int(r["status"].item()),
                                 "error_vs_oracle": errs(got, ref, x_ref, sd)}
        if cpu:
            res["cpu_baseline"] = {"value": 1.0 / t_or, "unit": "filter+sample calls/s",
                                   "cores": 1, "kind": "oracle",
                                   "sample": f"one sequential FP64 Kalman filter and RTS sample "
                                             f"(d={d}, T={N}) by the C oracle, {t_or:.2f} s",
                                   **host_info()}
        out[name] = res
    return out


def sampler_cpu_baseline(w, mf_dev, Pf_dev, dnc_steps: int = 512) -> dict:
    """The oracle's two samplers on the same filtering moments: the prefix-sum
    (RTS) sampler over the full series, the divide-and-conquer sampler over the
    first dnc_steps steps scaled to the full length (its work is linear in T)."""
    import numpy as np
    import oracle
    kw = w.oracle_kwargs()
    F, Q, b = kw["F"], kw["Q"], kw.get("b")
    mf = mf_dev.cpu().numpy()
    Pf = Pf_dev.cpu().numpy()
    mp = np.empty_like(mf)
    Pp = np.empty_like(Pf)
    mp[0], Pp[0] = kw["m0"], kw["P0"]
    mp[1:] = mf[:-1] @ F.T + (0.0 if b is None else b)
    Pp[1:] = F @ Pf[:-1] @ F.T + Q
    xi = np.random.default_rng(5).standard_normal(mf.shape)
    t0 = time.perf_counter()
    oracle.rts_sample(F, mf, Pf, mp, Pp, xi)
    t_rts = time.perf_counter() - t0
    n = min(dnc_steps, w.N)
    t0 = time.perf_counter()
    oracle.dnc_sample(F, Q, mf[:n], Pf[:n], xi[:n], b=b)
    t_dnc = (time.perf_counter() - t0) * w.N / n
    return {"prefix_sum": {"value": 1.0 / t_rts, "unit": "samples/s", "cores": 1,
                           "kind": "oracle",
                           "sample": f"one full RTS sample (T = {w.N}), {t_rts:.1f} s",
                           **host_info()},
            "divide_and_conquer": {"value": 1.0 / t_dnc, "unit": "samples/s", "cores": 1,
                                   "kind": "oracle",
                                   "sample": f"the first {n} steps of one sample, scaled by "
                                             f"{w.N}/{n}: {t_dnc:.1f} s per full sample",
                                   **host_info()}}


def progress(msg: str) -> None:
    """One line on stderr as each bench object starts, so a long run shows it is alive."""
    print(f"bench: {msg}", file=sys.stderr, flush=True)


def main() -> int:
    ap = argparse.ArgumentParser(description=__doc__)
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=30)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--repeats", type=int, default=5,
                    help="timed repeats of --steps steps; the headline is their median")
    ap.add_argument("--block", type=int, default=0, help="scan block size (0 = automatic)")
    ap.add_argument("--cpu-steps", type=int, default=2, help="oracle steps for cpu_baseline")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--roofline-kernel", default="filter_fold")
    ap.add_argument("--no-batched", action="store_true")
    ap.add_argument("--batched-steps", type=int, default=5)
    ap.add_argument("--no-adjoint", action="store_true")
    ap.add_argument("--no-gibbs", action="store_true")
    ap.add_argument("--gibbs-sweeps", type=int, default=200)
    ap.add_argument("--no-stoch-vol", action="store_true")
    ap.add_argument("--no-spatio-temporal", action="store_true")
    ap.add_argument("--no-lorenz", action="store_true")
    ap.add_argument("--no-samplers", action="store_true")
    ap.add_argument("--no-first-order", action="store_true")
    ap.add_argument("--no-poisson", action="store_true")
    ap.add_argument("--no-obs-lin", action="store_true")
    ap.add_argument("--no-sqrt", action="store_true")
    ap.add_argument("--eager", action="store_true",
                    help="time the eager launches only (no graph capture; for profiler runs)")
    ap.add_argument("--no-reuse", action="store_true")
    ap.add_argument("--copy-calibration", type=int, default=0, metavar="MIB",
                    help="after the bench, run 3 plain device copies of MIB MiB (a known-size "
                         "reference for the HBM byte counters)")
    args = ap.parse_args()

    world = int(os.environ.get("WORLD_SIZE", "1"))
    if args.gpus != 1 or world != 1:
        print(f"bench.py measures one GPU only (asked for --gpus {args.gpus}, WORLD_SIZE {world}): "
              "the sampler runs one chain per GPU and no multi-GPU path is built.",
              file=sys.stderr)
        return 2

    import torch
    from paper_2303_00301_amd import workloads as W
    from paper_2303_00301_amd import sampler as S
    from paper_2303_00301_amd import _lib

    dev = torch.device("cuda", 0)
    torch.cuda.set_device(dev)
    w = W.latent_field()
    N, d = w.N, w.dx
    B = args.block or auto_block(N, d)
    M = S.DeviceModel.from_workload(w, device=dev)
    y = torch.as_tensor(w.y, dtype=torch.float64, device=dev)
    x = torch.as_tensor(w.x_true, dtype=torch.float64, device=dev).contiguous()
    K, Wm, R = args.steps, args.warmup, args.repeats
    gen = torch.Generator(device=dev)
    gen.manual_seed(103)
    xi = torch.randn((R * K + Wm, 2, N, d), dtype=torch.float64, device=dev, generator=gen)
    un = torch.rand((R * K + Wm,), dtype=torch.float64, device=dev,
                    generator=gen).clamp_(min=1e-300)
    ws = S.Workspace(dev)

    # warm-up
    if Wm:
        S.mh_run(M, y, x, w.delta, w.order, xi[:Wm], un[:Wm], block=B, ws=ws)
    torch.cuda.synchronize()

    # R timed repeats of K steps each (the chain continues across repeats, with
    # fresh normals); the headline is the median repeat
    lib = _lib.load()
    fam = _lib.FAMILIES[args.roofline_kernel]
    _lib.check(lib.akf_timing_enable(fam, 8 * K * R + 16), "akf_timing_enable")
    ev0 = torch.cuda.Event(enable_timing=True)
    ev1 = torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    rep_ms, accs, n_bad = [], [], 0
    for r in range(R):
        sl = slice(Wm + r * K, Wm + (r + 1) * K)
        ev0.record()
        out = S.mh_run(M, y, x, w.delta, w.order, xi[sl], un[sl], block=B, ws=ws)
        ev1.record()
        torch.cuda.synchronize()
        rep_ms.append(ev0.elapsed_time(ev1))
        accs.append(out["accepted"].float().mean().item())
        n_bad += int((out["status"] != 0).sum().item())
    import ctypes as C
    n_l = C.c_int32()
    k_ms = C.c_double()
    _lib.check(lib.akf_timing_collect(C.byref(n_l), C.byref(k_ms)), "akf_timing_collect")
    lib.akf_timing_enable(-1, 0)

    acc_eager = sum(accs) / len(accs)
    eager_ms_step = sorted(rep_ms)[len(rep_ms) // 2] / K

    # Headline: the same K-step run captured once as a graph and replayed, with
    # fresh normals written into the captured buffers between replays (outside
    # the timed region).  First, one replay is checked against an eager run on
    # the same start and normals (same kernels: the results must be identical).
    xi_g = torch.empty((K, 2, N, d), dtype=torch.float64, device=dev)
    un_g = torch.empty((K,), dtype=torch.float64, device=dev)

    def refill():
        xi_g.normal_(generator=gen)
        un_g.uniform_(generator=gen).clamp_(min=1e-300)

    refill()
    x_cap = x.clone()
    if args.eager:
        rep_g, graph_ok, acc = rep_ms, None, acc_eager
        status_bad = n_bad
    S.mh_run(M, y, x_cap, w.delta, w.order, xi_g, un_g, block=B, ws=ws)  # warm the graph's shapes
    if not args.eager:
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            g_out = S.mh_run(M, y, x_cap, w.delta, w.order, xi_g, un_g, block=B, ws=ws)
        torch.cuda.synchronize()
        x_cap.copy_(x)
        graph.replay()
        x_eager = x.clone()
        e_out = S.mh_run(M, y, x_eager, w.delta, w.order, xi_g, un_g, block=B, ws=ws)
        torch.cuda.synchronize()
        graph_ok = bool(torch.equal(x_cap, x_eager) and
                        torch.equal(g_out["log_ratio"], e_out["log_ratio"]) and
                        torch.equal(g_out["accepted"], e_out["accepted"]))
        rep_g, accs, n_bad = [], [], 0
        for r in range(R):
            refill()
            torch.cuda.synchronize()
            ev0.record()
            graph.replay()
            ev1.record()
            torch.cuda.synchronize()
            rep_g.append(ev0.elapsed_time(ev1))
            accs.append(g_out["accepted"].float().mean().item())
            n_bad += int((g_out["status"] != 0).sum().item())
        acc = sum(accs) / len(accs)
        status_bad = n_bad
    ms_total = sorted(rep_g)[len(rep_g) // 2]
    ms_step = ms_total / K
    steps_s = 1000.0 / ms_step

    roof = None
    if n_l.value > 0:
        avg_ms = k_ms.value / n_l.value
        if args.roofline_kernel == "filter_fold":
            flops = fold_flops_per_launch(N, d, B)
        else:
            flops = float("nan")
        achieved = flops / (avg_ms * 1e-3) / 1e12
        roof = {"bound": "mfma", "achieved": achieved, "peak": PEAK_FP64_TFLOPS,
                "unit": "TFLOP/s", "frac": achieved / PEAK_FP64_TFLOPS,
                "traffic": measured_traffic(B) if args.roofline_kernel == "filter_fold" else None,
                "kernel": f"k_filter_fold<64> ({args.roofline_kernel})",
                "avg_launch_ms": avg_ms, "launches": n_l.value,
                "flops_per_launch": flops}

    progress(f"headline: {steps_s:.1f} steps/s")
    res = {
        "metric": METRIC,
        "value": steps_s,
        "unit": "steps/s",
        "n_gpus": 1,
        "steps": K,
        "warmup": Wm,
        "ms_per_step": ms_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64",
        "data": "synthetic",
        "config": {"workload": f"latent_field_d{d}_T{N}: periodic-grid Gaussian dynamics, "
                               f"Student-t(3, 0.5) at 32 sites, order-2 proposal, one chain",
                   "d_x": d, "T": N, "chains": 1, "order": w.order, "delta": w.delta,
                   "scan_block": B},
        "time_steps_per_s": steps_s * N,
        "repeats": R,
        "timing": ("median of the eager repeats (HIP events; --eager)" if args.eager else
                   "median of the repeats of one captured K-step graph replayed with fresh "
                   "normals (HIP events); eager launches of the same run beside it"),
        "repeat_ms_per_step": [m / K for m in rep_g],
        "graph_replay_equals_eager": graph_ok,
        "eager_ms_per_step": eager_ms_step,
        "eager_repeat_ms_per_step": [m / K for m in rep_ms],
        "eager_acceptance": acc_eager,
        "acceptance": acc,
        "rejected_by_status": status_bad,
        "roofline": roof,
    }
    if not args.no_batched:
        progress("batched ...")
        res["batched"] = bench_batched(torch, S, W, _lib, args.batched_steps, dev,
                                       not args.no_cpu_baseline)
    if not args.no_adjoint:
        progress("adjoint ...")
        res["adjoint"] = bench_adjoint(torch, S, W, _lib, 5, dev, not args.no_cpu_baseline)
    if not args.no_gibbs:
        progress("gibbs ...")
        res["gibbs"] = bench_gibbs(torch, S, W, _lib, args.gibbs_sweeps, dev,
                                   not args.no_cpu_baseline)
    if not args.no_stoch_vol:
        progress("stoch_vol ...")
        res["stoch_vol"] = bench_stoch_vol(torch, S, W, _lib, 20, dev,
                                           0 if args.no_cpu_baseline else 20)
    if not args.no_spatio_temporal:
        progress("spatio_temporal ...")
        res["spatio_temporal"] = bench_spatio_temporal(
            torch, S, W, _lib, 100, dev, 0 if args.no_cpu_baseline else 100)
    if not args.no_samplers:
        progress("samplers ...")
        res["samplers"] = bench_samplers(torch, S, W, _lib, 5, dev, not args.no_cpu_baseline)
    if not args.no_obs_lin:
        progress("obs_linearisation ...")
        res["obs_linearisation"] = bench_obs_linearisation(
            torch, S, W, _lib, 20, dev, 0 if args.no_cpu_baseline else 1)
    if not args.no_sqrt:
        progress("sqrt ...")
        res["sqrt_filter"] = bench_sqrt(torch, S, W, _lib, 10, dev, not args.no_cpu_baseline)
    if not args.no_poisson:
        progress("poisson ...")
        res["poisson"] = bench_poisson(torch, S, W, _lib, 50, dev,
                                       0 if args.no_cpu_baseline else 20)
    if not args.no_first_order:
        progress("first_order ...")
        res["first_order"] = bench_first_order(torch, S, W, _lib, 50, dev,
                                               0 if args.no_cpu_baseline else 1)
    if not args.no_reuse:
        progress("reuse_order2 ...")
        res["reuse_order2"] = bench_reuse(torch, S, W, _lib, 30, dev)
    if not args.no_lorenz:
        progress("nonlinear ...")
        res["nonlinear"] = bench_lorenz(torch, S, W, _lib, 20, dev,
                                        0 if args.no_cpu_baseline else 10)
    if not args.no_cpu_baseline and args.cpu_steps > 0:
        progress("cpu_baseline ...")
        res["cpu_baseline"] = cpu_baseline(w, args.cpu_steps)
        if "reuse_order2" in res:
            # the oracle's plain order-2 step is the same computation on the same workload
            res["reuse_order2"]["cpu_baseline"] = dict(res["cpu_baseline"])
    if args.copy_calibration > 0:
        n = args.copy_calibration * (1 << 20) // 8
        src = torch.ones(n, dtype=torch.float64, device=dev)
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        res["copy_calibration_bytes"] = n * 8
    print(json.dumps(res), flush=True)
    return 0


if __name__ == "__main__":
    sys.exit(main())
