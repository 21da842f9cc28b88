"""Benchmark: reduced-Hessian HVPs per second on the 10k-bus synthetic grid.

One step = the full dense reduced Hessian (n_p = 2,799 directions) computed
through the C ABI in k = 256 direction blocks, which share a call's launches,
with every input already resident on the GPU.  The timed region brackets
exactly `--steps` steps with device synchronisations.  Prints one JSON line.

Roofline: a step is one call, a sequence of kernels (the tree path).  Its
algorithmic HBM bytes are (10 n_x + 5 n_p) * 8 per direction (every
intermediate written and read once, W read twice, H written) plus the factor
entries of the four triangular sweeps (12 bytes each), the per-incidence
coefficients and G_p; achieved GB/s = those bytes / the average call's duration
from HIP events recorded on the launch stream.  Peak: 8 TB/s (MI355X HBM3E).

The CPU baseline runs the FP64 oracle (SuperLU solves and sparse products)
on the same grid: the whole Hessian split over every host core, one process
per core, with the one-core rate beside it.
"""
import argparse
import hashlib
import json
import os
import sys
import time
from pathlib import Path

ROOT = Path(__file__).resolve().parent
sys.path.insert(0, str(ROOT))

import numpy as np  # noqa: E402

PEAK_HBM_GBS = 8000.0
# per path the measured memory traffic and the sources it depends on: the
# kernels, the planner that lays out what they read, and their shared headers
TRAFFIC = {
    "block_kernel": ("block_kernel_10k_hbm_traffic.txt", ("device.hip", "rh_internal.h", "sparse_lu.cpp")),
    "tree path": ("tree_path_hbm_traffic.txt", ("tree.hip", "tree.cpp", "tree.h", "tree_device.h", "sparse_lu.cpp")),
}


def sources_digest(kernel):
    """SHA-256 over a path's sources (TRAFFIC), in name order."""
    h = hashlib.sha256()
    for name in sorted(TRAFFIC[kernel][1]):
        f = ROOT / "paper_2201_00241_amd" / "csrc" / name
        h.update(f.name.encode())
        h.update(f.read_bytes())
    return h.hexdigest()


def measured_traffic(kernel):
    """HBM bytes per launch of the headline's path from the committed counter
    summary, or None if its sources changed since it was measured."""
    f = ROOT / "profiles" / TRAFFIC[kernel][0]
    if not f.exists():
        return None
    kv = {}
    for line in f.read_text().splitlines():
        if ":" in line and not line.startswith(("#", " ", "|")):
            key, val = line.split(":", 1)
            kv[key.strip()] = val.strip()
    if kv.get("sources_sha256") != sources_digest(kernel):
        return None
    try:
        return float(kv["traffic_bytes_per_launch"])
    except (KeyError, ValueError):
        return None


def algorithmic_bytes_per_launch(rep, g, kb):
    """Algorithmic HBM bytes of one launch over kb directions (FP64)."""
    n_x, n_p = rep["n_x"], rep["n_p"]
    per_dir = (10 * n_x + 5 * n_p) * 8
    factors = 2 * (rep["nnz_l"] + rep["nnz_u"]) * 12  # L, U, U^T, L^T sweeps
    tape = 2 * g.n_branch * (5 * 8 + 4) + g.n_bus * 8 * 3
    gp = 2 * (n_x + 2 * g.n_branch * 2) * 12
    return per_dir * kb + factors + tape + gp


def mean_bytes_per_launch(rep, g, n_p, k):
    """Average of algorithmic_bytes_per_launch over the ceil(n_p / k) launches
    of a full Hessian (the last one carries n_p mod k directions)."""
    kbs = [min(k, n_p - j0) for j0 in range(0, n_p, k)]
    return sum(algorithmic_bytes_per_launch(rep, g, kb) for kb in kbs) / len(kbs)


def host_cpu():
    """CPU model and the number of cores this process may use: the affinity
    set, capped by the cgroup CPU quota when one is set, and at 16 (the host
    share of one GPU on a shared box)."""
    model = "unknown"
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                model = line.split(":", 1)[1].strip()
                break
    except OSError:
        pass
    try:
        n = len(os.sched_getaffinity(0))
    except AttributeError:
        n = os.cpu_count() or 1
    quota = None
    try:
        q, period = open("/sys/fs/cgroup/cpu.max").read().split()[:2]
        if q != "max":
            quota = float(q) / float(period)
    except (OSError, ValueError):
        pass
    if quota is not None:
        n = min(n, max(1, int(quota)))
    return model, max(1, min(n, 16)), quota


def _oracle_worker(config, lo, hi, barrier, out):
    """One process of the multi-core baseline: its own oracle set-up (Newton,
    SuperLU, lambda), then identity columns [lo, hi) of the full Hessian as
    one block, timed from a barrier shared with the other workers."""
    sys.path.insert(0, str(ROOT))
    import gridgen
    from oracle import solve

    s = solve(gridgen.config_grid(config, 0))
    n_p = s.o.n_p
    W = np.zeros((n_p, hi - lo))
    W[np.arange(lo, hi), np.arange(hi - lo)] = 1.0
    barrier.wait()
    t0 = time.perf_counter()
    s.hvp(W)
    out.put((hi - lo, time.perf_counter() - t0))


_THREAD_VARS = ("OMP_NUM_THREADS", "OPENBLAS_NUM_THREADS", "MKL_NUM_THREADS", "BLIS_NUM_THREADS")


def cpu_baseline(config, g, k, budget_s=12.0):
    """The oracle on the same workload: one core for up to budget_s, then the
    whole Hessian split over every host core (one process per core, each with
    its own SuperLU); the headline figure is the multi-core rate."""
    import multiprocessing as mp

    from oracle import solve

    t0 = time.perf_counter()
    s = solve(g)
    setup = time.perf_counter() - t0
    n_p = s.o.n_p
    done = 0
    t1 = time.perf_counter()
    while done < n_p and time.perf_counter() - t1 < budget_s:
        kb = min(k, n_p - done)
        W = np.zeros((n_p, kb))
        W[np.arange(done, done + kb), np.arange(kb)] = 1.0
        s.hvp(W)
        done += kb
    el = time.perf_counter() - t1
    one_core = done / el
    model, cores, quota = host_cpu()
    # contiguous column ranges, one per process; every process runs one
    # thread (the variables are set before the children import numpy)
    step = -(-n_p // cores)
    ranges = [(lo, min(n_p, lo + step)) for lo in range(0, n_p, step)]
    ctx = mp.get_context("spawn")
    barrier = ctx.Barrier(len(ranges))
    q = ctx.Queue()
    saved = {v: os.environ.get(v) for v in _THREAD_VARS}
    for v in _THREAD_VARS:
        os.environ[v] = "1"
    try:
        procs = [ctx.Process(target=_oracle_worker, args=(config, lo, hi, barrier, q))
                 for lo, hi in ranges]
        for p in procs:
            p.start()
        res = [q.get(timeout=600) for _ in procs]
        for p in procs:
            p.join()
    finally:
        for v, val in saved.items():
            if val is None:
                os.environ.pop(v, None)
            else:
                os.environ[v] = val
    cols = sum(r[0] for r in res)
    wall = max(r[1] for r in res)
    return {
        "value": cols / wall, "unit": "HVP/s", "cores": len(ranges), "kind": "oracle",
        "cpu_model": model, "cgroup_cpu_quota": quota,
        "one_core": {"value": one_core, "unit": "HVP/s", "cores": 1,
                     "sample": f"{done} of {n_p} identity directions in k={k} blocks ({el:.1f} s)"},
        "sample": f"all {n_p} identity directions of the full Hessian, split into {len(ranges)} "
                  f"contiguous column ranges of up to {step}, one per process (SciPy SuperLU, one "
                  f"thread each, each range one block), {wall:.2f} s from a common start; each "
                  f"process's Newton+LU+lambda set-up ({setup:.1f} s on one core) not included",
    }


def cpu_baseline_tracking(steps=3, seed=5):
    """The oracle's tracking update (power flow, reduced gradient, reduced
    Hessian, Cholesky, projected update) on one host core, for the first
    steps of the 1,000-bus trajectory that run_tracking times on the GPU."""
    import gridgen
    from oracle import powerflow as opf
    from oracle import tracking as otr

    g = gridgen.config_grid("c1", 0)
    orc = opf.Oracle(g)
    p0 = orc.p0()
    npv = orc.npv  # parameter order: Pg at PV buses, v_ref, v at PV buses
    volt = np.arange(p0.size) >= npv
    lo = np.where(volt, 0.94, 0.0)
    hi = np.where(volt, 1.06, 2.0 * np.maximum(p0, 0.1))
    ramp = np.where(volt, 0.002, 0.01)
    Pd, Qd = gridgen.load_trajectory(g, steps=60, seed=seed)
    gg = g.copy()
    p, x, ms = np.clip(p0, lo, hi), None, []
    for t in range(steps):
        gg.Pd, gg.Qd = Pd[t].copy(), Qd[t].copy()
        t0 = time.perf_counter()
        s_, _, _, d_, _ = otr.step(gg, p, x0=x)
        ms.append(1e3 * (time.perf_counter() - t0))
        x, p = s_.x, otr.project(p, d_, lo, hi, ramp)
    return {"update_ms_median": float(np.median(ms)), "cores": 1, "kind": "oracle",
            "sample": f"the first {steps} updates of the 1,000-bus tracking trajectory"}


def refined_bytes_per_direction(n_x, n_p, passes_z, passes_psi):
    """Algorithmic bytes of one direction in the refined mode, counting every
    pass made: per FP32 pass (the first solve or a correction) the FP32
    intermediate of the first sweep and the FP32 correction written and read
    (2 x 2 x 4 n_x), the FP64 residual and the FP64 solution read and written
    (2 x 2 x 8 n_x); outside the passes the right-hand side B and Z, -Y_x, Psi
    (8 n_x each) and W twice, Y_p, H (5 n_p x 8)."""
    per_pass = (2 * 2 * 4 + 2 * 2 * 8) * n_x
    return (passes_z + passes_psi) * per_pass + 4 * 8 * n_x + 5 * 8 * n_p


def refined_launch_bytes(rep, g, kb, passes_z, passes_psi, nnz_gx):
    """Per launch: the directions' bytes plus, per pass, the FP32 factor
    entries of both sweeps (8 bytes) and the FP64 residual matrix (12 bytes),
    and once the tape and G_p."""
    n_x, n_p = rep["n_x"], rep["n_p"]
    per_pass_factors = (rep["nnz_l"] + rep["nnz_u"]) * 8 + nnz_gx * 12
    tape = 2 * g.n_branch * (5 * 8 + 4) + g.n_bus * 8 * 3
    gp = 2 * (n_x + 2 * g.n_branch * 2) * 12
    return (kb * refined_bytes_per_direction(n_x, n_p, passes_z, passes_psi)
            + (passes_z + passes_psi) * per_pass_factors + tape + gp)


def _parallel_networks(ctx, grids):
    """Create and solve one network per grid on a few host threads (the C ABI
    allows distinct handles on different threads)."""
    from concurrent.futures import ThreadPoolExecutor

    from paper_2201_00241_amd import rh

    def make(g):
        n = rh.Network(ctx, g)
        n.solve(1e-13, 30)
        return n

    with ThreadPoolExecutor(max_workers=min(8, len(grids))) as ex:
        return list(ex.map(make, grids))


def run_refined(net, g, H, k, steps, warmup, stream):
    """The refined FP32 mode on the headline workload: HVP/s, per-column
    refinement figures and the roofline fraction over every pass made."""
    import torch

    from paper_2201_00241_amd import rh

    n_p = net.n_p
    sptr = stream.cuda_stream
    H64 = H.clone()
    tile = net.autotune(prec=rh.RH_FP32_REFINED)
    for _ in range(warmup):
        net.reduced_hessian_device(H, k_block=k, stream=sptr, prec=rh.RH_FP32_REFINED)
    torch.cuda.synchronize()
    net.ctx.set_timing(1)
    net.report()
    r0, r1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    r0.record(stream)
    for _ in range(steps):
        net.reduced_hessian_device(H, k_block=k, stream=sptr, prec=rh.RH_FP32_REFINED)
    r1.record(stream)
    torch.cuda.synchronize()
    rep = net.report()
    net.ctx.set_timing(0)
    ms = r0.elapsed_time(r1) / steps
    fig = net.refinement_report(n_p)
    pz = 1.0 + float(np.mean(fig["steps_z"]))
    pp = 1.0 + float(np.mean(fig["steps_psi"]))
    per = -(-n_p // max(1, rep["last_launches"] // steps))  # directions of a launch (blocks may share one)
    kbs = [min(per, n_p - j0) for j0 in range(0, n_p, per)]
    bytes_launch = sum(refined_launch_bytes(rep, g, kb, pz, pp, rep["nnz_gx"]) for kb in kbs) / len(kbs)
    avg_launch_ms = rep["last_kernel_ms"] / rep["last_launches"]
    achieved = bytes_launch / (avg_launch_ms / 1e3) / 1e9
    dev = float((H - H64).abs().max() / H64.abs().max())
    H.copy_(H64)
    return {
        "value": n_p / (ms / 1e3), "unit": "HVP/s", "ms_per_step": ms, "k": k,
        "dirs_per_group": rep["dirs_per_group"], "max_rel_dev_from_fp64": dev,
        "tuned_shape": tile,
        "passes_per_solve": {"z": pz, "psi": pp},
        "corrections_histogram": {"z": np.bincount(fig["steps_z"]).tolist(),
                                  "psi": np.bincount(fig["steps_psi"]).tolist()},
        "max_backward_error": {"z": float(fig["berr_z"].max()), "psi": float(fig["berr_psi"].max())},
        "roofline": {"bound": "hbm", "achieved": achieved, "peak": PEAK_HBM_GBS, "unit": "GB/s",
                     "frac": achieved / PEAK_HBM_GBS, "kernel": "tree path" if rep["dirs_per_group"] == 16 else "refined_kernel",
                     "avg_launch_ms": avg_launch_ms, "algorithmic_bytes_per_launch": bytes_launch},
        "what": "same workload, FP32 sweeps with FP64 residual refinement (each direction stops "
                "at a backward error of 1e-13 or after 4 corrections)",
    }


def run_batch(instances, steps, warmup, config="c3"):
    """Operating points of one grid (loads perturbed by up to 10 %), each with
    128 Gaussian directions, in one launch per step; FP64 and refined."""
    import torch

    import gridgen
    from paper_2201_00241_amd import rh

    base = gridgen.config_grid(config, 0)
    ctx = rh.Context(0)
    t0 = time.perf_counter()
    nets = _parallel_networks(ctx, [gridgen.perturb_loads(base, seed=5000 + i) for i in range(instances)])
    setup_s = time.perf_counter() - t0
    k = 128
    Ws = [torch.from_numpy(np.ascontiguousarray(gridgen.directions(n.n_p, k, 7000 + i).T)).cuda()
          for i, n in enumerate(nets)]
    HWs = [torch.empty_like(W) for W in Ws]
    stream = torch.cuda.current_stream()
    out = {}
    HW64 = None
    for name, prec in (("fp64", rh.RH_FP64), ("refined_fp32", rh.RH_FP32_REFINED)):
        # the batched launch recorded once as a graph, replayed every step
        batch = ctx.batch(nets, Ws, HWs, prec=prec)
        for _ in range(warmup):
            batch.launch(stream.cuda_stream)
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(stream)
        for _ in range(steps):
            batch.launch(stream.cuda_stream)
        e1.record(stream)
        torch.cuda.synchronize()
        ms = e0.elapsed_time(e1) / steps
        info = batch.info()
        batch.close()
        # one eager batched call (host-side work list, one launch) beside it
        ctx.set_timing(1)
        ctx.report()
        t0 = time.perf_counter()
        ctx.hvp_batch_device(nets, Ws, HWs, stream=stream.cuda_stream, prec=prec)
        torch.cuda.synchronize()
        eager_wall_ms = (time.perf_counter() - t0) * 1e3
        rep = ctx.report()
        ctx.set_timing(0)
        out[name] = {"value": len(nets) * k / (ms / 1e3), "unit": "HVP/s", "ms_per_step": ms,
                     "launch": "graph replay (rh_batch_launch)",
                     "dirs_per_group": info["dirs_per_group"], "workgroups": info["workgroups"],
                     "eager_kernel_ms": rep["last_kernel_ms"], "eager_wall_ms": eager_wall_ms}
        if HW64 is None:
            HW64 = [h.clone() for h in HWs]
        else:
            out[name]["max_rel_dev_from_fp64"] = max(
                float((h - g).abs().max() / g.abs().max()) for h, g in zip(HWs, HW64))
    for n in nets:
        n.close()
    ctx.close()
    out.update({
        "workload": f"{len(nets)} operating points of a {base.n_bus}-bus grid (loads x U(0.9, 1.1)) "
                    f"x {k} Gaussian directions, one launch per step",
        "n_x": nets[0].n_x, "n_p": nets[0].n_p, "setup_s": setup_s,
    })
    return out


def run_serving(n_peak=120, n_run=300, seed=11):
    """Poisson arrivals over resident 1k, 10k and 70k networks (4 operating
    points each); requests for 1, 16 or 128 directions or the full Hessian,
    FP64 or refined.  The peak is the closed-loop rate of the same mix; the
    arrival times are scaled so that the offered rate (requests / last
    arrival) is exactly 0.8 x peak."""
    import gridgen
    from paper_2201_00241_amd import rh
    from paper_2201_00241_amd.serving import Request, Server, latency_summary

    ctx = rh.Context(0)
    grids, keys = [], []
    for name in ("c1", "c2", "c3"):
        base = gridgen.config_grid(name, 0)
        for i in range(4):
            grids.append(gridgen.perturb_loads(base, seed=9000 + i))
            keys.append(f"{name}/{i}")
    t0 = time.perf_counter()
    nets = dict(zip(keys, _parallel_networks(ctx, grids)))
    setup_s = time.perf_counter() - t0
    rng = np.random.default_rng(seed)

    def make(n_req):
        reqs = []
        for i in range(n_req):
            key = keys[rng.integers(len(keys))]
            k = int(rng.choice([1, 16, 128, 0], p=[0.3, 0.3, 0.3, 0.1]))
            prec = rh.RH_FP64 if rng.random() < 0.5 else rh.RH_FP32_REFINED
            W = None if k == 0 else rng.standard_normal((nets[key].n_p, k))
            reqs.append(Request(rid=i, key=key, k=k, W=W, prec=prec))
        return reqs

    srv = Server(ctx, nets, max_inflight=3, dirs_per_launch=4096, block=256,
                 mem_budget_bytes=128 << 30, keep_results=False)
    srv.run(make(12))  # warm-up
    t0 = time.perf_counter()
    closed = srv.run(make(n_peak))
    peak = len(closed) / (time.perf_counter() - t0)
    reqs = make(n_run)
    gaps = rng.exponential(1.0, n_run)
    arr = np.cumsum(gaps)
    arr *= n_run / (0.8 * peak) / arr[-1]  # offered rate n_run / arr[-1] = 0.8 peak
    for r, a in zip(reqs, arr):
        r.arrival = float(a)
    t0 = time.perf_counter()
    done = srv.run(reqs)
    wall = time.perf_counter() - t0
    ok = [r for r in done if r.error is None]
    hvps = sum((r.k if r.k else nets[r.key].n_p) for r in ok)
    lat = latency_summary(ok)
    for n in nets.values():
        n.close()
    ctx.close()
    return {
        "p50_ms": lat["p50_ms"], "p99_ms": lat["p99_ms"], "mean_ms": lat["mean_ms"],
        "requests": len(done), "failed": len(done) - len(ok),
        "offered_rate_req_s": n_run / float(arr[-1]), "peak_req_s": peak,
        "offered_fraction_of_peak": n_run / float(arr[-1]) / peak,
        "served_req_s": len(ok) / wall, "served_hvp_s": hvps / wall,
        "latency": "scheduled arrival to the completion event of the request's last block",
        "workload": "Poisson arrivals over 1k/10k/70k-bus grids, 4 load-perturbed operating points "
                    "each; k in {1,16,128} (0.3 each) or the full Hessian (0.1); FP64 or refined "
                    "FP32 (0.5 each)",
        "setup_s": setup_s,
    }


def _tracking_limits(net):
    """Bounds and per-minute ramp limits of the controls: generator outputs in
    [0, 2 max(Pg0, 0.1)] moving at most 0.01 pu per step, voltage set-points in
    [0.94, 1.06] moving at most 0.002 pu per step."""
    _, _, _, pk = net.index_maps()
    p0 = net.get_parameters()
    volt = pk == 1
    lo = np.where(volt, 0.94, 0.0)
    hi = np.where(volt, 1.06, 2.0 * np.maximum(p0, 0.1))
    ramp = np.where(volt, 0.002, 0.01)
    return lo, hi, ramp


def run_tracking(steps=60, seed=5):
    """Real-time tracking (Sec. 6.3, eq. (qp_rto); Table 3): one update per
    minute of a synthetic load trajectory on the 1,000-bus grid, each update =
    power flow at the new loads (device Newton, warm-started), then Step 1
    (reduced gradient and full reduced Hessian) and Step 2 (dense Cholesky
    solve of H d = -g and the projected update of p), all on the GPU.  Also
    single updates on the 10,000-bus grid."""
    import torch

    import gridgen
    from paper_2201_00241_amd import rh

    out = {}
    ctx = rh.Context(0)
    g = gridgen.config_grid("c1", 0)
    net = rh.Network(ctx, g)
    lo, hi, ramp = _tracking_limits(net)
    p_start = np.clip(net.get_parameters(), lo, hi)
    net.set_parameters(p_start)
    Pd, Qd = gridgen.load_trajectory(g, steps=steps, seed=seed)
    net.solve_device()
    tile = net.autotune()  # launch shape of H, outside the timed steps
    rows = []
    for t in range(steps):
        net.set_loads(Pd[t], Qd[t])
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        it, _ = net.solve_device()
        t1 = time.perf_counter()
        info = net.tracking_step_device(lo=lo, hi=hi, ramp=ramp)
        t2 = time.perf_counter()
        rows.append((1e3 * (t1 - t0), 1e3 * (t2 - t1), info, it))
    solve_ms = np.array([r[0] for r in rows])
    step_ms = np.array([r[1] for r in rows])
    hess_ms = np.array([r[2]["ms_gradient"] + r[2]["ms_hessian"] for r in rows])
    chol_ms = np.array([r[2]["ms_solve"] for r in rows])
    out["grid_1k"] = {
        "steps": steps, "n_p": net.n_p, "tuned_shape": tile,
        "median_ms": {"power_flow": float(np.median(solve_ms)),
                      "step1_gradient_hessian": float(np.median(hess_ms)),
                      "step2_cholesky_solve": float(np.median(chol_ms)),
                      "update_wall": float(np.median(step_ms)),
                      "total_wall": float(np.median(solve_ms + step_ms))},
        "max_total_wall_ms": float(np.max(solve_ms + step_ms)),
        "newton_iters_median": float(np.median([r[3] for r in rows])),
        "shifted_steps": int(sum(r[2]["tau"] > 0 for r in rows)),
        "workload": "1,000-bus grid, 60 one-minute load steps (common swing 3%, per-bus noise 0.5%, "
                    "seed 5), Pg ramp 0.01 pu/min, voltage ramp 0.002 pu/min",
    }
    net.close()
    # single updates at 10,000 buses (base loads)
    g2 = gridgen.config_grid("c2", 0)
    net2 = rh.Network(ctx, g2)
    lo2, hi2, ramp2 = _tracking_limits(net2)
    net2.set_parameters(np.clip(net2.get_parameters(), lo2, hi2))
    net2.solve_device()
    net2.autotune()
    r2 = []
    for t in range(3):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        net2.solve_device()
        t1 = time.perf_counter()
        info = net2.tracking_step_device(lo=lo2, hi=hi2, ramp=ramp2)
        t2 = time.perf_counter()
        r2.append((1e3 * (t1 - t0), 1e3 * (t2 - t1), info))
    out["grid_10k"] = {
        "n_p": net2.n_p, "updates": len(r2),
        "median_ms": {"power_flow": float(np.median([r[0] for r in r2])),
                      "step1_gradient_hessian": float(np.median([r[2]["ms_gradient"] + r[2]["ms_hessian"]
                                                                 for r in r2])),
                      "step2_cholesky_solve": float(np.median([r[2]["ms_solve"] for r in r2])),
                      "update_wall": float(np.median([r[1] for r in r2]))},
    }
    net2.close()
    ctx.close()
    out["paper_table3_context"] = {"case": "PEGASE1354 (n_p = 519)", "hardware": "V100 vs Xeon Gold 6140",
                                   "gpu_s": {"step1": 0.05, "step2": 0.05, "total": 0.10},
                                   "cpu_s": {"step1": 1.41, "step2": 0.81, "total": 2.22}}
    return out


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--config", default="c2")
    ap.add_argument("--k", type=int, default=256)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-serving", action="store_true")
    ap.add_argument("--no-batch", action="store_true")
    ap.add_argument("--no-refined", action="store_true")
    ap.add_argument("--no-tracking", action="store_true")
    ap.add_argument("--workload", default="hessian",
                    choices=["hessian", "batch", "serving", "tracking"],
                    help="hessian: full reduced Hessian (the headline metric, with the batched "
                         "and serving figures attached); batch: only the operating points of "
                         "one grid in one launch; serving: only the Poisson request mix")
    ap.add_argument("--instances", type=int, default=32)
    ap.add_argument("--copy-probe", type=int, default=0,
                    help="only run a device-to-device copy of this many bytes, 10 times "
                         "(reference for scaling HBM traffic counters)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(json.dumps({"error": "this benchmark runs on one GPU; --gpus must be 1 "
                                   "(direction blocks are independent and would shard across "
                                   "GPUs by block, which is not implemented)"}))
        sys.exit(2)

    import torch

    if args.copy_probe:
        n = args.copy_probe // 8
        src = torch.ones(n, dtype=torch.float64, device="cuda")
        dst = torch.empty_like(src)
        for _ in range(10):
            dst.copy_(src)
        torch.cuda.synchronize()
        print(json.dumps({"copy_probe_bytes_read": n * 8, "copy_probe_bytes_written": n * 8,
                          "launches": 10}), flush=True)
        return

    import gridgen
    from paper_2201_00241_amd import rh

    assert torch.cuda.is_available(), "bench needs a GPU"
    torch.cuda.set_device(0)
    if args.workload == "batch":
        print(json.dumps(run_batch(args.instances, args.steps, args.warmup)), flush=True)
        return
    if args.workload == "serving":
        print(json.dumps(run_serving()), flush=True)
        return
    if args.workload == "tracking":
        print(json.dumps(run_tracking()), flush=True)
        return
    g = gridgen.config_grid(args.config, 0)
    ctx = rh.Context(0)
    net = rh.Network(ctx, g)
    t0 = time.perf_counter()
    net.solve(1e-13, 30)
    setup_s = time.perf_counter() - t0
    n_p = net.n_p
    k = min(args.k, n_p)
    H = torch.empty((n_p, n_p), dtype=torch.float64, device="cuda")
    stream = torch.cuda.current_stream()
    sptr = stream.cuda_stream
    # launch shape (directions per workgroup, sweep schedule) from the tuner;
    # the headline keeps k = 256 directions per block
    t0 = time.perf_counter()
    tile = net.autotune()
    tune_s = time.perf_counter() - t0
    print(f"# tuned shape: {tile} ({tune_s:.1f} s)", file=sys.stderr, flush=True)

    for _ in range(args.warmup):
        net.reduced_hessian_device(H, k_block=k, stream=sptr)
    torch.cuda.synchronize()

    ctx.set_timing(True)
    net.report()  # open a fresh timing window
    step_ms = []
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(args.steps + 1)]
    torch.cuda.synchronize()
    t_start = time.perf_counter()
    ev[0].record(stream)
    for i in range(args.steps):
        net.reduced_hessian_device(H, k_block=k, stream=sptr)
        ev[i + 1].record(stream)
    torch.cuda.synchronize()
    wall = time.perf_counter() - t_start
    trep = net.report()  # launch durations of the timed region
    ctx.set_timing(False)
    for i in range(args.steps):
        step_ms.append(ev[i].elapsed_time(ev[i + 1]))
    total_ms = ev[0].elapsed_time(ev[-1])
    ms_per_step = total_ms / args.steps
    value = n_p * args.steps / (total_ms / 1e3)
    print(f"# headline: {value:.0f} HVP/s, {ms_per_step:.3f} ms per Hessian", file=sys.stderr, flush=True)

    # the tuner's own launch size (outside the timed region)
    torch.cuda.synchronize()
    e_a, e_b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    net.reduced_hessian_device(H, k_block=0, stream=sptr)
    e_a.record(stream)
    for _ in range(3):
        net.reduced_hessian_device(H, k_block=0, stream=sptr)
    e_b.record(stream)
    torch.cuda.synchronize()
    tuned_ms = e_a.elapsed_time(e_b) / 3

    # one more step with in-kernel phase stamps (outside the timed region)
    ctx.set_timing(2)
    net.reduced_hessian_device(H, k_block=k, stream=sptr)
    torch.cuda.synchronize()
    prep = net.report()
    ctx.set_timing(0)

    rep = trep
    launches = trep["last_launches"]
    avg_launch_ms = trep["last_kernel_ms"] / launches
    # directions of a launch: the k blocks of a Hessian may share one
    dirs = -(-n_p // max(1, launches // args.steps))
    bytes_launch = mean_bytes_per_launch(rep, g, n_p, dirs)
    achieved = bytes_launch / (avg_launch_ms / 1e3) / 1e9
    kernel = "tree path" if rep["dirs_per_group"] == 16 else "block_kernel"
    traffic = measured_traffic(kernel)
    phase_names = ["spmul", "L", "U", "projection", "Ut", "Lt", "spmuladd"]
    out = {
        "metric": "reduced-Hessian HVPs/sec at 10k buses (k=256) vs plain; p50/p99 latency",
        "value": value,
        "unit": "HVP/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_per_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64",
        "data": "synthetic",
        "config": {
            "workload": f"full reduced Hessian of a {g.n_bus}-bus synthetic grid "
                        f"({g.n_branch} branches, {g.n_gen} generators) in k={k} blocks",
            "n_x": rep["n_x"], "n_p": n_p, "k": k,
            "loading_factor": g.meta.get("alpha"),
            "mean_pq_load_pu": float(np.mean(g.Pd[g.bus_type == gridgen.PQ])),
            "launches_per_step": launches // args.steps,
            "dirs_per_group": rep["dirs_per_group"],
            "levels_l": rep["levels_l"], "levels_u": rep["levels_u"],
            "nnz_l": rep["nnz_l"], "nnz_u": rep["nnz_u"],
            "steps_l": rep["steps_l"], "steps_u": rep["steps_u"],
            "tuned_shape": {**tile, "tune_s": tune_s,
                            "source": ["defaults", "measured", "cache"][tile["source"]]},
        },
        "phase_us": dict(zip(phase_names, [round(v, 2) for v in prep["phase_us"]])),
        "latency_ms": {"p50": float(np.percentile(step_ms, 50)),
                       "p99": float(np.percentile(step_ms, 99)),
                       "what": "one full reduced Hessian"},
        "roofline": {
            "bound": "hbm", "achieved": achieved, "peak": PEAK_HBM_GBS, "unit": "GB/s",
            "frac": achieved / PEAK_HBM_GBS, "traffic": traffic,
            "traffic_unit": "HBM bytes per launch (rocprofv3 FETCH_SIZE + WRITE_SIZE, copy-scaled)",
            "kernel": kernel, "avg_launch_ms": avg_launch_ms,
            "algorithmic_bytes_per_launch": bytes_launch,
        },
        "setup_s": setup_s,
        "wall_s": wall,
        "tuned_k_full_hessian": {"k": tile["k"], "ms_per_step": tuned_ms, "value": n_p / (tuned_ms / 1e3),
                                 "what": "the same full Hessian with the tuner's launch size"},
    }
    # per-phase roofline fractions: each phase's algorithmic bytes (a launch's directions)
    # over its mean time per workgroup
    n_x = rep["n_x"]
    ph_bytes = {"L": 2 * n_x * dirs * 8 + rep["nnz_l"] * 12, "U": 2 * n_x * dirs * 8 + rep["nnz_u"] * 12,
                "Ut": 2 * n_x * dirs * 8 + rep["nnz_u"] * 12, "Lt": 2 * n_x * dirs * 8 + rep["nnz_l"] * 12,
                "projection": 2 * (n_x + n_p) * dirs * 8}
    out["phase_roofline_frac"] = {
        p: round(b / (out["phase_us"][p] * 1e-6) / 1e9 / PEAK_HBM_GBS, 4)
        for p, b in ph_bytes.items() if out["phase_us"].get(p, 0) > 0}
    if not args.no_refined:
        out["refined_fp32"] = run_refined(net, g, H, k, args.steps, args.warmup, stream)
        print(f"# refined: {out['refined_fp32']['value']:.0f} HVP/s", file=sys.stderr, flush=True)
    net.close()
    ctx.close()
    if not args.no_batch:
        out["batch"] = run_batch(args.instances, max(2, args.steps // 4), 1)
        print(f"# batch: {out['batch']['fp64']['value']:.0f} HVP/s", file=sys.stderr, flush=True)
    if not args.no_tracking:
        out["tracking"] = run_tracking()
        tr = out["tracking"]["grid_1k"]["median_ms"]
        print(f"# tracking 1k: {tr['total_wall']:.1f} ms per update (power flow {tr['power_flow']:.1f}, "
              f"step 1 {tr['step1_gradient_hessian']:.2f}, step 2 {tr['step2_cholesky_solve']:.2f})",
              file=sys.stderr, flush=True)
    if not args.no_serving:
        out["serving"] = run_serving()
        print(f"# serving: p50 {out['serving']['p50_ms']:.1f} ms p99 {out['serving']['p99_ms']:.1f} ms",
              file=sys.stderr, flush=True)
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(args.config, g, k)
        out["cpu_baseline"]["tracking"] = cpu_baseline_tracking()
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
