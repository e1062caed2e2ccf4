"""Benchmark: masked LDDMM on the atlas-sized workload, one MI355X.

One step = one full registration: 3-level pyramid (4x, 2x, 1x), T = 10 time
steps, 200 iterations per level, on the 264 x 160 x 228 atlas-like pair
(50 um voxels, sparse target) -- every step of the hot path (flow, warp,
residual and energy, adjoint transport, Jacobian, body force, K smoothing,
update, guard, pyramid transfer) runs in the HIP library.

value = voxel-timestep updates per second = sum over levels of
(user voxels x T x iterations) / wall seconds, inputs resident in HBM.

Usage: python bench.py [--gpus 1] [--steps K] [--warmup W] [--no-cpu-baseline]
"""

from __future__ import annotations

import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
# Algorithmic bytes per voxel and launch, one weighted channel (FP32):
#  forward step : read v 12, read u0 12, gather J0 4, write u0 12, write J0_t 4
#  backward step: read v 12, read u1 12, write u1 12, gather r 4, read J0_t 4, write b 12
#  K (all five passes together): read b 12, write K b 12; update: read v 12, K b 12, write v 12
#  each FFT pass on its own: read and write its operand once (x inverse: + v read and write)
ALG_BYTES = {"forward": 44.0, "backward": 56.0, "fft_x": 24.0, "fft_y": 24.0, "fft_zK": 24.0,
             "fft_yinv": 24.0, "fft_xinv_update": 36.0}
K_CHAIN = ("fft_x", "fft_y", "fft_zK", "fft_yinv", "fft_xinv_update")
K_CHAIN_ALG_BYTES = 60.0    # K as one round trip (24) + the update (36), per voxel-timestep
SWEEP_CLASSES = ("forward", "backward", "fft_x", "fft_y", "fft_zK", "fft_yinv",
                 "fft_xinv_update", "forward_edge", "backward_edge")
B_ALG_PATH = 162.0          # per voxel-timestep per iteration, whole path

LEVELS = 3
T = 10
FLAGS = 0                   # library flags of the atlas workload (atlas-rk4: LDDMM_FLAG_RK4)
INTEGRATOR = "euler"        # the oracle's name for the same flow integrator
ITERS = (200, 200, 200)
SPACING = 0.05              # mm: the 264 x 160 x 228 grid is the atlas at 50 um
ALPHA, GAMMA, SIGMA = 0.02, 1.0, 1.0
STEP = 0.02
GUARD = False               # plain fixed-step descent: every slot is a full iteration


def log(msg):
    print(msg, file=sys.stderr, flush=True)


def workload_config():
    integ = "first-order semi-Lagrangian" if FLAGS == 0 else "fourth-order Runge-Kutta"
    return {"workload": "atlas-like 264x160x228 masked LDDMM (Mask-LDDMM channel), "
                        f"3-level pyramid 4x/2x/1x, T={T} ({integ} departure points), "
                        "200 iterations/level",
            "integrator": INTEGRATOR,
            "grid": [264, 160, 228], "comp_grid_finest": [280, 160, 240],
            "levels": LEVELS, "timesteps": T, "iters_per_level": list(ITERS),
            "spacing_mm": SPACING, "alpha": ALPHA, "gamma": GAMMA, "sigma": SIGMA,
            "step": STEP, "guard": GUARD, "weights": [1.0, 0.0]}


def attainable_bandwidth(torch, L, nbytes=None, reps=10):
    """HBM bandwidth the library's copy kernel reaches (read + write bytes / time),
    timed with events on its stream: the ceiling a streaming kernel can expect in
    practice, beside the published peak.  The copy is the size of the finest-level
    velocity (COPY_FLOATS), the same copy the counter calibration uses."""
    nbytes = 4 * COPY_FLOATS if nbytes is None else nbytes
    src = torch.empty(nbytes // 4, dtype=torch.float32, device="cuda").fill_(1.0)
    dst = torch.empty_like(src)
    stream = torch.cuda.current_stream()
    L.lddmm_copy(src, dst, stream=stream)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    e0.record(stream)
    for _ in range(reps):
        L.lddmm_copy(src, dst, stream=stream)
    e1.record(stream)
    torch.cuda.synchronize()
    gbs = 2.0 * nbytes * reps / (e0.elapsed_time(e1) * 1e-3) / 1e9
    del src, dst
    return gbs


def kernel_name(cls, tunables, rk4, nch=1):
    """The kernel a profile class launches at the finest atlas level (as the rocprofv3
    summaries name it), given the launch-shape choice."""
    b = lambda x: "true" if x else "false"
    if cls == "forward":
        zm = tunables.get("fwd_tiles", 1792) > 0
        return f"k_forward<{nch}, false, false, {b(rk4)}, {b(zm)}>"
    if cls == "backward":
        if tunables.get("staged_min_blocks", 2048) <= 3200:   # 3200 staged blocks at 280x160x240
            return f"k_backward_staged<{nch}, true, {b(rk4)}>"
        return f"k_backward<{nch}, true, false, true, {b(rk4)}>"
    return {"fft_x": "k_fft_x_fwd", "fft_y": "k_fft_y<*, false>", "fft_zK": "k_fft_z_K",
            "fft_yinv": "k_fft_y<*, true>", "fft_xinv_update": "k_fft_x_inv"}.get(cls, cls)


def last_accepted_D(tr):
    """Masked SSD term D of the current iterate at the end: the D of the last
    accepted trial (a rejected or stopped slot's D is not the iterate's)."""
    ok = np.where((tr[:, 6] == 1) & np.isfinite(tr[:, 2]))[0]
    return float(tr[ok[-1], 2]) if len(ok) else float("nan")


def work_units(shape):
    """sum over levels of user voxels x T x iterations."""
    nz, ny, nx = shape
    tot = 0
    for li in range(LEVELS):
        s = 2 ** (LEVELS - 1 - li)
        n = (-(-nx // s)) * (-(-ny // s)) * (-(-nz // s))
        tot += n * T * ITERS[li]
    return tot


def _oracle_iterations(args):
    """One worker of the CPU baseline: plain oracle iterations of the coarsest level
    until the time budget is used (at least 2).  Returns (iterations, seconds)."""
    pair_arrays, budget_s = args
    from oracle import lddmm as O
    M0, M1, MI0, MI1 = pair_arrays
    prm = O.Params(alpha=ALPHA, gamma=GAMMA, sigma=SIGMA, T=T, step=STEP, spacing=SPACING,
                   integrator=INTEGRATOR)
    prob = O.Problem(M0, M1, MI0, MI1)
    J0u, J1u = prob.channels()
    grids = O.level_grids(M0.shape, LEVELS)
    Pf = grids[-1]["P"]
    J0 = [O.pad_to(f, Pf) for f in J0u]
    J1 = [O.pad_to(f, Pf) for f in J1u]
    for _ in range(LEVELS - 1):
        J0 = [O.downsample2(f) for f in J0]
        J1 = [O.downsample2(f) for f in J1]
    h = SPACING * grids[0]["h"]
    v = np.zeros((T, 3) + grids[0]["P"])
    t0 = time.perf_counter()
    iters = 0
    st = O.energy_terms(v, J0, J1, prm, h)
    while True:
        gV, _ = O.gradient_V(v, st, prm, h)
        v = v - prm.step * gV
        st = O.energy_terms(v, J0, J1, prm, h)
        iters += 1
        if iters >= 2 and time.perf_counter() - t0 > budget_s:
            break
    return iters, time.perf_counter() - t0


def cpu_baseline(pair, budget_s=20.0):
    """The FP64 oracle as it stands on a bounded sample: one worker process per host
    core (at most 16), each running plain iterations of the coarsest level of the
    same workload for the time budget; the value is the workers' combined
    voxel-timesteps per second."""
    import multiprocessing as mp
    try:
        cores = len(os.sched_getaffinity(0))
    except AttributeError:
        cores = os.cpu_count() or 1
    workers = max(1, min(16, cores))
    grids = __import__("oracle.lddmm", fromlist=["level_grids"]).level_grids(pair.shape, LEVELS)
    g = grids[0]
    arrays = (pair.M0, pair.M1, pair.MI0, pair.MI1)
    env = {k: os.environ.get(k) for k in ("OMP_NUM_THREADS", "OPENBLAS_NUM_THREADS",
                                          "MKL_NUM_THREADS")}
    for k in env:
        os.environ[k] = "1"                    # one thread per worker process
    try:
        ctx = mp.get_context("spawn")
        t0 = time.perf_counter()
        with ctx.Pool(workers) as pool:
            out = pool.map(_oracle_iterations, [(arrays, budget_s)] * workers)
        wall = time.perf_counter() - t0
    finally:
        for k, val in env.items():
            if val is None:
                os.environ.pop(k, None)
            else:
                os.environ[k] = val
    nz, ny, nx = g["N"]
    units = sum(nx * ny * nz * T * it for it, _ in out)
    secs = max(sec for _, sec in out)
    return {"value": units / secs, "unit": "voxel-timestep/s", "cores": workers,
            "host_cores_available": cores, "kind": "oracle",
            "sample": f"{workers} worker processes (one thread each), each running plain "
                      f"iterations (forward + backward + K + update) of the coarsest level "
                      f"({nx}x{ny}x{nz} user voxels, computational grid "
                      f"{g['P'][2]}x{g['P'][1]}x{g['P'][0]}, T={T}) for about {budget_s:.0f} s: "
                      f"{sum(it for it, _ in out)} iterations in all, {secs:.1f} s per worker "
                      f"({wall:.1f} s wall); FP64 NumPy oracle, numpy.fft"}


def _short_name(name):
    """Kernel name without namespaces and argument list."""
    import re
    name = name.replace("(anonymous namespace)::", "").replace("lddmm::", "")
    return re.sub(r"\(.*", "", name)


def _kernel_rows(db):
    """Per-dispatch rows (name, grid threads, duration ns, counter, value) of a rocprofv3 DB."""
    import re
    import sqlite3
    c = sqlite3.connect(db)
    out = []
    try:
        q = "select kernel_name, grid_size, duration, counter_name, value from counters_collection"
        for name, grid, dur, cn, val in c.execute(q):
            out.append((_short_name(name), grid, dur, cn, val))
    except sqlite3.Error:
        pass
    if not out:
        q = "select name, grid_x*grid_y*grid_z, duration from kernels"
        for name, grid, dur in c.execute(q):
            out.append((_short_name(name), grid, dur, None, None))
    return out


def _split_levels(items):
    """Split the dispatches of one (kernel, grid) group at their largest duration gap
    when durations span more than 4x (the same launch shape at two pyramid levels)."""
    items = sorted(items, key=lambda r: r[0])
    d = [r[0] for r in items]
    if len(d) < 2 or d[-1] <= 4 * d[0]:
        return [("", items)]
    k = max(range(1, len(d)), key=lambda i: d[i] / max(d[i - 1], 1))
    return [(" (short)", items[:k]), (" (long)", items[k:])]


def summarize_profile(db, out_path, command):
    """Write a text summary of a rocprofv3 DB: per (kernel, grid) calls, mean/min/max
    duration and, for counter runs, mean counter value per dispatch (KiB for
    FETCH_SIZE / WRITE_SIZE).  Returns {(kernel, grid, level tag): (calls, mean ns, mean counter)}."""
    from collections import defaultdict
    groups = defaultdict(list)
    for name, grid, dur, cn, val in _kernel_rows(db):
        groups[(name, grid, cn)].append((dur, val))
    rows = []
    for (name, grid, cn), items in groups.items():
        for tag, part in _split_levels(items):
            durs = [p[0] for p in part]
            vals = [p[1] for p in part if p[1] is not None]
            rows.append((name, grid, tag, cn, len(part), sum(durs), min(durs), max(durs),
                         sum(vals) / len(vals) if vals else None))
    tot = sum(r[5] for r in rows)
    lines = [f"# rocprofv3 summary of: {command}", f"# database: {os.path.basename(db)}",
             f"# total kernel time {tot / 1e6:.3f} ms over {sum(r[4] for r in rows)} dispatches",
             "# grid = launch threads; (short)/(long): one launch shape at two problem sizes",
             f"{'kernel':58s} {'grid':>18s} {'calls':>6s} {'avg_us':>9s} {'min_us':>8s} "
             f"{'max_us':>8s} {'share':>6s} {'counter':>10s} {'avg/dispatch':>14s}"]
    out = {}
    for name, grid, tag, cn, n, s, mn, mx, cv in sorted(rows, key=lambda r: -r[5]):
        cnt = f"{cv:14.1f}" if cv is not None else ""
        lines.append(f"{name[:58]:58s} {str(grid) + tag:>18s} {n:6d} {s / n / 1e3:9.2f} "
                     f"{mn / 1e3:8.2f} {mx / 1e3:8.2f} {100 * s / tot:5.1f}% "
                     f"{(cn or ''):>10s} {cnt}")
        out[(name, grid, tag)] = (n, s / n, cv)
    with open(out_path, "w") as f:
        f.write("\n".join(lines) + "\n")
    return out


def library_sources_sha():
    """SHA-256 of what builds the measured kernels (the sweeps and the FFT passes):
    their sources and compiler flags (paths left out), to tell whether stored
    counters describe them."""
    import hashlib
    from paper_1605_02060_amd import build as B
    hsh = hashlib.sha256()
    for rel in ("paper_1605_02060_amd/csrc/flow.hip", "paper_1605_02060_amd/csrc/fft.hip",
                "paper_1605_02060_amd/csrc/device.h", "paper_1605_02060_amd/csrc/internal.h",
                "include/lddmm.h"):
        with open(os.path.join(ROOT, rel), "rb") as f:
            hsh.update(rel.encode())
            hsh.update(f.read())
    for src in ("flow.hip", "fft.hip"):
        hsh.update(" ".join(f for f in B.flags_for(src) if not os.path.isabs(f)).encode())
    return hsh.hexdigest()


TRAFFIC_FILE = os.path.join(ROOT, "profiles", "traffic_atlas_finest.json")


def stored_traffic(kernel):
    """HBM bytes per launch of `kernel` at the finest level from the committed counter runs,
    or None when the counters were taken on other kernel sources."""
    try:
        with open(TRAFFIC_FILE) as f:
            t = json.load(f)
    except (OSError, ValueError):
        return None
    if t.get("source_sha") != library_sources_sha():
        return None
    k = t.get("kernels", {}).get(kernel)
    return None if k is None else k["fetch_bytes"] + k["write_bytes"]


# Calibration: the bandwidth probe's copy of the finest-level velocity (k_copy of
# 3 T |P| floats) reads and writes exactly this many bytes.
COPY_FLOATS = 3 * T * 280 * 160 * 240
FINEST_VOXELS = 280 * 160 * 240


def compute_traffic(fetch_db, write_db, out_path):
    """Bytes per finest-level launch of the forward and backward sweep classes from two
    rocprofv3 counter runs of the bench command (FETCH_SIZE, then WRITE_SIZE, KiB per
    dispatch), each scaled by what that counter reads for the copy kernel of known size."""
    import re
    from collections import defaultdict

    def per_kernel(db, counter):
        rows = defaultdict(list)
        for name, grid, dur, cn, val in _kernel_rows(db):
            if cn == counter:
                rows[(name, grid)].append((dur, val))
        return rows

    out = {"source_sha": library_sources_sha(), "grid": [280, 160, 240],
           "calibration": f"k_copy of the finest-level velocity ({COPY_FLOATS} floats = "
                          f"{4 * COPY_FLOATS} bytes read and written)", "kernels": {}}
    factors = {}
    per = {}
    for tag, db, counter in (("fetch", fetch_db, "FETCH_SIZE"), ("write", write_db, "WRITE_SIZE")):
        rows = per_kernel(db, counter)
        # the probe's copies are the group of the longest ones
        allc = [(d, v) for (name, grid), items in rows.items() if name == "k_copy"
                for d, v in items]
        if not allc:
            raise SystemExit(f"no k_copy dispatch in {db}")
        dmax = max(d for d, v in allc)
        copy = [v for d, v in allc if d >= 0.7 * dmax]
        factors[tag] = 4.0 * COPY_FLOATS / (1024.0 * sum(copy) / len(copy))
        per[tag] = rows
    out["fetch_factor"], out["write_factor"] = factors["fetch"], factors["write"]
    # finest-level dispatches of each class.  A launch-shape group (split where
    # one shape runs at two pyramid levels) is at the finest level when its mean
    # counter value is at least 0.3 of the class's largest: levels differ 8x in
    # voxels, the kernel variants of a class (first step, map-only steps) at most
    # about 2x in bytes per voxel, so the coarser levels fall below and a variant
    # that never runs on the finest grid drops out.  Of a variant's finest-level
    # groups the one with the most dispatches is taken (the timed steps, not the
    # autotuner's trials of other shapes).  Grids alone do not tell the levels
    # apart: plane-marching launches size their grid by planes and runs, so a
    # coarser level can launch more blocks.
    # one kernel per class, as the profile classes of the bench line count them
    classes = {"forward": r"^void k_forward<\d+, false, false,",
               "backward": r"^void k_backward(_staged<\d+, true,|<\d+, true, false, true,)",
               "fft_x": r"^void k_fftc?_x_fwd<", "fft_y": r"^void k_fftc?_y<[\d, ]+, false>",
               "fft_zK": r"^void k_fftc?_(z_K|zK)<", "fft_yinv": r"^void k_fftc?_y<[\d, ]+, true>",
               "fft_xinv_update": r"^void k_fftc?_x_inv<"}
    for cls, pat in classes.items():
        tot = {"fetch": [], "write": []}
        durs = []
        for tag in ("fetch", "write"):
            parts = [(name, part) for (name, grid), items in per[tag].items()
                     if re.match(pat, name)
                     for sub, part in _split_levels([(d, v) for d, v in items])]
            if not parts:
                continue
            mean_v = [sum(v for d, v in part) / len(part) for name, part in parts]
            top = max(mean_v)
            for name in sorted({name for name, part in parts}):
                cand = [part for (n2, part), m in zip(parts, mean_v) if n2 == name and m >= 0.3 * top]
                if not cand:
                    continue
                part = max(cand, key=len)
                tot[tag] += [v * 1024.0 * factors[tag] for d, v in part]
                if tag == "fetch":
                    durs += [d for d, v in part]
        if tot["fetch"] and tot["write"]:
            f = sum(tot["fetch"]) / len(tot["fetch"])
            w = sum(tot["write"]) / len(tot["write"])
            out["kernels"][cls] = {"launches": len(tot["fetch"]), "fetch_bytes": f, "write_bytes": w,
                                   "fetch_bytes_per_voxel": f / FINEST_VOXELS,
                                   "write_bytes_per_voxel": w / FINEST_VOXELS,
                                   "mean_us_under_counters": sum(durs) / len(durs) / 1e3}
    with open(out_path, "w") as fh:
        json.dump(out, fh, indent=1)
    print(json.dumps(out["kernels"], indent=1))


BATCH_ITERS = 100


def bench_batched(args):
    """16 pairs of uneven size (64..160 per axis), T = 10, 100 fixed-step iterations
    each, one level: batched grouped launches against 16 sequential single-pair runs,
    launch shapes from the autotuner (tuned outside the timed region)."""
    import torch
    from paper_1605_02060_amd import lddmm as L
    from paper_1605_02060_amd import synth
    from paper_1605_02060_amd import tune

    L.load()
    assert torch.cuda.is_available(), "bench needs a GPU"
    dims = synth.batched_dims()
    pairs, units = [], 0
    for k in range(len(dims)):
        p = synth.batched_pair(k, dims)
        tt = lambda a: torch.as_tensor(a, device="cuda")
        pairs.append({"M0": tt(p.M0), "M1": tt(p.M1), "spacing": SPACING})
        units += p.M0.size * T * BATCH_ITERS
        log(f"pair {k} {tuple(int(d) for d in dims[k])} generated")
    prm = L.Params(alpha=ALPHA, gamma=GAMMA, sigma=SIGMA, T=T, n_levels=1, iters=(BATCH_ITERS,),
                   step=STEP, guard=GUARD, weight=(1.0, 0.0))
    t0 = time.perf_counter()
    choice = tune.autotune(pairs, prm, verbose=True)
    log(f"autotune {time.perf_counter() - t0:.1f} s: "
        f"{ {tune.NAMES[w]: v for w, v in choice.items()} }")
    wss = [L.workspace(tuple(d["M0"].shape), prm, SPACING) for d in pairs]
    vs = [torch.zeros((T, 3) + L.lddmm_comp_grid(tuple(d["M0"].shape), prm, 0, SPACING),
                      dtype=torch.float32, device="cuda") for d in pairs]

    def batched():
        for v in vs:
            v.zero_()
        return L.lddmm_register_batched(pairs, prm, vs=vs, wss=wss, want_phi=False)

    def sequential():
        out = []
        for d, v, ws in zip(pairs, vs, wss):
            v.zero_()
            out.append(L.lddmm_register(d["M0"], d["M1"], params=prm, spacing=SPACING, v=v,
                                        ws=ws, want_phi=False))
        return out

    for w in range(max(args.warmup, 1)):
        batched()
        sequential()
        torch.cuda.synchronize()
        log(f"warmup {w} done")
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        res, code = batched()
    torch.cuda.synchronize()
    tb = (time.perf_counter() - t0) / args.steps
    log(f"batched {tb:.3f} s per step")
    t0 = time.perf_counter()
    for _ in range(args.steps):
        seq = sequential()
    torch.cuda.synchronize()
    ts = (time.perf_counter() - t0) / args.steps
    log(f"sequential {ts:.3f} s per step")
    for r, s in zip(res, seq):
        assert torch.equal(r["v"], s["v"]), "batched and sequential results differ"
    final_D = [float(r["trace"][-1, 2]) for r in res]
    out = {
        "metric": "voxel-timestep updates/s (flow+adjoint+K); time to target masked SSD",
        "value": units / tb,
        "unit": "voxel-timestep/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": tb * 1e3,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic (seeded blob pairs scaled to each grid, plane-wave warps)",
        "config": {"workload": "batched: 16 masked LDDMM pairs, grids rng(4) in 64..160 per "
                               "axis, T=10, 100 iterations each, one level",
                   "grids_xyz": [[int(x) for x in d] for d in dims], "timesteps": T,
                   "iters": BATCH_ITERS, "spacing_mm": SPACING, "step": STEP, "guard": GUARD,
                   "tunables": {tune.NAMES[w]: v for w, v in choice.items()}},
        "sequential": {"value": units / ts, "ms_per_step": ts * 1e3},
        "batched_speedup": ts / tb,
        "path_roofline": {"alg_bytes_per_voxel_timestep": B_ALG_PATH,
                          "frac": units / tb * B_ALG_PATH / 1e9 / HBM_PEAK_GBS},
        "final_masked_ssd": final_D,
        "status": int(code),
    }
    print(json.dumps(out), flush=True)


HIST_CALLS = 100            # histogram matches per step of the histmatch workload
HIST_BINS, HIST_POINTS = 32, 8
# Algorithmic bytes per voxel of each histogram-matching pass (FP32 image + mask):
#  range (in-mask min / max): read I, M of both images     8 per voxel of either image
#  count (bins + point table): read I, M of both images    8 per voxel of either image
#  apply (map): read I0, M0, write the matched image      12 per template voxel
HIST_ALG_BYTES = {"hist_range": 8.0, "hist_count": 8.0, "hist_apply": 12.0}


def hist_cpu_baseline(pair, budget_s=15.0):
    """The oracle's histogram matching of the same pair, repeated for about budget_s."""
    from oracle import histmatch as H
    t0 = time.perf_counter()
    calls = 0
    while True:
        H.histogram_match(pair.I0, pair.M0, pair.I1, pair.M1, HIST_BINS, HIST_POINTS)
        calls += 1
        if time.perf_counter() - t0 > budget_s:
            break
    dt = time.perf_counter() - t0
    return {"value": calls * (pair.M0.size + pair.M1.size) / dt, "unit": "voxel/s", "cores": 1,
            "kind": "oracle",
            "sample": f"{calls} full histogram matches of the same 264x160x228 pair in {dt:.1f} s; "
                      "NumPy (float32 bins, FP64 table and map), single-threaded"}


def bench_histmatch(args):
    """Image-LDDMM preprocessing at the atlas size (Methods, Preprocessing): the
    atlas-like template image, masked, histogram-matched (32 bins, 8 quantile
    points) to the masked sparse target image, both 264 x 160 x 228."""
    import torch
    from paper_1605_02060_amd import lddmm as L
    from paper_1605_02060_amd import synth

    L.load()
    assert torch.cuda.is_available(), "bench needs a GPU"
    log("generating atlas-like pair ...")
    pair = synth.config_pair("atlas")
    tt = lambda a: torch.as_tensor(a, device="cuda")
    I0, M0, I1, M1 = tt(pair.I0.astype(np.float32)), tt(pair.M0), tt(pair.I1.astype(np.float32)), \
        tt(pair.M1)
    ns, nr = pair.M0.size, pair.M1.size
    ws = torch.empty(L.lddmm_histogram_match_workspace_size(pair.shape, pair.shape, HIST_BINS),
                     dtype=torch.uint8, device="cuda")

    def step():
        for _ in range(HIST_CALLS):
            res = L.lddmm_histogram_match(I0, M0, I1, M1, HIST_BINS, HIST_POINTS, ws=ws,
                                          want_points=True, want_counts=False)
        return res

    for w in range(max(args.warmup, 1)):
        step()
        torch.cuda.synchronize()
        log(f"warmup {w} done")
    classes = ("hist_range", "hist_count", "hist_apply")
    L.lddmm_profile_begin(sum(1 << L.PROF_CLASSES.index(c) for c in classes), 0)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        out, pts, _ = step()
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    prof = L.lddmm_profile_end()
    calls = HIST_CALLS * args.steps
    value = calls * (ns + nr) / elapsed
    per = {}
    for c in classes:
        avg_ms = prof[c]["ms"] / max(prof[c]["launches"], 1)
        vox = prof[c]["voxels"] / max(prof[c]["launches"], 1)
        per[c] = {"avg_us": 1e3 * avg_ms, "voxels": vox,
                  "GBs": HIST_ALG_BYTES[c] * vox / (avg_ms * 1e-3) / 1e9}
    dominant = max(classes, key=lambda c: per[c]["avg_us"])
    achieved = per[dominant]["GBs"]
    cpu = None
    if not args.no_cpu_baseline:
        log("cpu baseline (oracle) ...")
        cpu = hist_cpu_baseline(pair)
    pts = pts.cpu().numpy()
    res = {
        "metric": "histogram-matched voxels/s (Image-LDDMM preprocessing)",
        "value": value,
        "unit": "voxel/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": 1e3 * elapsed / args.steps,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32 bins, f64 table and map",
        "data": "synthetic (seeded atlas-like template, sparse Poisson-labelled warped target)",
        "config": {"workload": f"histogram matching of the masked 264x160x228 atlas-like template "
                               f"image to the masked sparse target image, {HIST_BINS} bins, "
                               f"{HIST_POINTS} quantile points; {HIST_CALLS} matches per step",
                   "grid": [264, 160, 228], "bins": HIST_BINS, "points": HIST_POINTS,
                   "calls_per_step": HIST_CALLS},
        "roofline": {"bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": achieved / HBM_PEAK_GBS, "traffic": None,
                     "kernel": {"hist_range": "k_hist_range_part + k_hist_range_final",
                                "hist_count": "k_hist_count + k_hist_sum + k_hist_table",
                                "hist_apply": "k_hist_apply"}[dominant],
                     "alg_bytes_per_voxel": HIST_ALG_BYTES[dominant],
                     "avg_launch_ms": per[dominant]["avg_us"] / 1e3,
                     "voxels_per_launch": per[dominant]["voxels"]},
        "passes": per,
        "call_us": 1e6 * elapsed / calls,
        "points": {"template": list(pts[0]), "target": list(pts[1])},
        "cpu_baseline": cpu,
    }
    print(json.dumps(res), flush=True)


ALIGN_SLOTS = (100, 100)    # rigid, then affine descent slots per step
ALIGN_STEP = 1.0
# Algorithmic bytes per target voxel of one MSE/gradient pass: read the target
# image 4, gather the template 4 (each template voxel once near the identity).
ALIGN_ALG_BYTES = 8.0


def align_cpu_baseline(pair, budget_s=15.0):
    """The oracle's MSE-and-gradient evaluation (one descent slot) on the same
    full-size masks, repeated for about budget_s (at least once)."""
    from oracle import align as A
    S = A.identity_map(pair.shape, SPACING, pair.shape, SPACING)
    t0 = time.perf_counter()
    slots = 0
    while True:
        A.mse_and_grad(S, pair.M0, SPACING, pair.M1, SPACING)
        slots += 1
        if time.perf_counter() - t0 > budget_s:
            break
    dt = time.perf_counter() - t0
    return {"value": slots * pair.M1.size / dt, "unit": "voxel-slot/s", "cores": 1,
            "kind": "oracle",
            "sample": f"{slots} MSE + gradient evaluations (one descent slot each) of the "
                      f"264x160x228 masks in {dt:.1f} s; FP64 NumPy, single-threaded"}


def bench_align(args):
    """Mask-Rigid then Mask-Affine pre-alignment (Methods, Registration) of the
    264 x 160 x 228 atlas-like template mask to the sparse target's mask at
    50 um: 100 rigid and 100 affine descent slots per step."""
    import torch
    from paper_1605_02060_amd import lddmm as L
    from paper_1605_02060_amd import synth

    L.load()
    assert torch.cuda.is_available(), "bench needs a GPU"
    log("generating atlas-like pair ...")
    pair = synth.config_pair("atlas")
    M0 = torch.as_tensor(pair.M0, device="cuda")
    M1 = torch.as_tensor(pair.M1, device="cuda")
    n1 = pair.M1.size
    ws = torch.empty(L.load().lddmm_align_workspace_size(ctypes_grid(L, pair.shape)),
                     dtype=torch.uint8, device="cuda")

    def step():
        Sr, tr_r = L.lddmm_align(M0, M1, L.ALIGN_RIGID, ALIGN_SLOTS[0], ALIGN_STEP,
                                 template_spacing=SPACING, target_spacing=SPACING, ws=ws)
        Sa, tr_a = L.lddmm_align(M0, M1, L.ALIGN_AFFINE, ALIGN_SLOTS[1], ALIGN_STEP, affine=Sr,
                                 template_spacing=SPACING, target_spacing=SPACING, ws=ws)
        return Sa, tr_r, tr_a

    for w in range(max(args.warmup, 1)):
        step()
        torch.cuda.synchronize()
        log(f"warmup {w} done")
    L.lddmm_profile_begin(1 << L.PROF_CLASSES.index("align"), 0)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        Sa, tr_r, tr_a = step()
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    prof = L.lddmm_profile_end()["align"]
    slots = (ALIGN_SLOTS[0] + 1 + ALIGN_SLOTS[1] + 1) * args.steps
    value = slots * n1 / elapsed
    avg_ms = prof["ms"] / max(prof["launches"], 1)
    achieved = ALIGN_ALG_BYTES * n1 / (avg_ms * 1e-3) / 1e9
    cpu = None
    if not args.no_cpu_baseline:
        log("cpu baseline (oracle) ...")
        cpu = align_cpu_baseline(pair)
    tr_r, tr_a = tr_r.cpu().numpy(), tr_a.cpu().numpy()
    out = {
        "metric": "alignment voxel-slots/s (MSE + gradient + guard per target voxel)",
        "value": value,
        "unit": "voxel-slot/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": 1e3 * elapsed / args.steps,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32 samples, f64 sums and maps",
        "data": "synthetic (seeded atlas-like template mask, sparse Poisson-labelled target mask)",
        "config": {"workload": "Mask-Rigid then Mask-Affine pre-alignment of the 264x160x228 "
                               "atlas-like mask pair at 50 um, 100 + 100 descent slots",
                   "grid": [264, 160, 228], "spacing_mm": SPACING, "slots": list(ALIGN_SLOTS),
                   "step": ALIGN_STEP},
        "roofline": {"bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": achieved / HBM_PEAK_GBS, "traffic": None,
                     "kernel": "k_align_partials", "alg_bytes_per_voxel": ALIGN_ALG_BYTES,
                     "avg_launch_ms": avg_ms, "launches": prof["launches"],
                     "voxels_per_launch": n1},
        "slot_us": 1e6 * elapsed / slots,
        "mse": {"start": float(tr_r[0, 0]), "after_rigid": float(np.nanmin(tr_r[:, 0])),
                "after_affine": float(np.nanmin(tr_a[:, 0]))},
        "cpu_baseline": cpu,
    }
    print(json.dumps(out), flush=True)


MASK_CALLS = 20             # target mask + surface distances per step
MASK_TAU, MASK_OPEN, MASK_CLOSE = 0.1, 0.05, 0.125   # threshold; 50 um and 125 um balls
# Algorithmic HBM bytes per voxel of each call (FP32 inputs and outputs; the
# bit-packed intermediates are 1/8 byte per voxel and pass):
#  target mask      : read the image 4, write the mask 4
#  surface distance : read both masks 8; per direction write the column distances 4
#                     (the z pass reads them only at surface voxels): 8 + 2 * 4
MASK_ALG_BYTES = {"target_mask": 8.0, "surface_distance": 16.0}
# The x + y distance pass writes the column distances of both directions; how many rows of a
# column it looks at depends on the masks, so its rate is given in bytes.
MASK_XY_BYTES = 8.0


def masks_image(pair):
    """A dense image of the atlas shape with foreground grains and holes."""
    rng = np.random.default_rng(7)
    I = pair.I0 * (1.0 + 0.2 * rng.standard_normal(pair.shape))
    I[rng.random(pair.shape) > 0.999] = 1.0
    I[rng.random(pair.shape) > 0.999] = 0.0
    return I.astype(np.float32)


def masks_cpu_baseline(pair, I, budget_s=15.0):
    """The oracle's target mask and surface distances of the same inputs,
    repeated for about budget_s (at least once)."""
    from oracle import masks as K
    t0 = time.perf_counter()
    calls = 0
    while True:
        M1 = K.target_mask(I, MASK_TAU, MASK_OPEN, MASK_CLOSE, SPACING)
        K.surface_distances(pair.M0 > 0, M1, SPACING)
        calls += 1
        if time.perf_counter() - t0 > budget_s:
            break
    dt = time.perf_counter() - t0
    return {"value": calls * I.size / dt, "unit": "voxel/s", "cores": 1, "kind": "oracle",
            "sample": f"{calls} target masks + surface distances of the 264x160x228 grid in "
                      f"{dt:.1f} s; NumPy shifts and scipy's k-d tree, single-threaded"}


def bench_masks(args):
    """Mask generation and evaluation at the atlas size (Methods, Mask Generation;
    Evaluation): the target mask by threshold, 50 um opening and 125 um closing,
    then the Hausdorff and median surface distances to the template mask."""
    import torch
    from paper_1605_02060_amd import lddmm as L
    from paper_1605_02060_amd import synth

    L.load()
    assert torch.cuda.is_available(), "bench needs a GPU"
    log("generating atlas-like pair ...")
    pair = synth.config_pair("atlas")
    I = torch.as_tensor(masks_image(pair), device="cuda")
    M0 = torch.as_tensor(pair.M0, device="cuda")
    n = pair.M0.size
    ws = torch.empty(L.load().lddmm_masks_workspace_size(ctypes_grid(L, pair.shape)),
                     dtype=torch.uint8, device="cuda")

    def step():
        for _ in range(MASK_CALLS):
            M1 = L.lddmm_target_mask(I, MASK_TAU, MASK_OPEN, MASK_CLOSE, spacing=SPACING, ws=ws)
            d = L.lddmm_surface_distance(M0, M1, spacing=SPACING, ws=ws)
        return d

    for w in range(max(args.warmup, 1)):
        step()
        torch.cuda.synchronize()
        log(f"warmup {w} done")
    # live HIP events: the library's own around its y-pass launches (the OTHER
    # class), torch's on the launch stream around whole calls
    L.lddmm_profile_begin(1 << L.PROF_CLASSES.index("other"), 0)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        d = step()
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    ypass = L.lddmm_profile_end()["other"]
    per = {}
    M1 = L.lddmm_target_mask(I, MASK_TAU, MASK_OPEN, MASK_CLOSE, spacing=SPACING, ws=ws)
    stream = torch.cuda.current_stream()
    for name in ("target_mask", "surface_distance"):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        e0.record(stream)
        for _ in range(MASK_CALLS):
            if name == "target_mask":
                L.lddmm_target_mask(I, MASK_TAU, MASK_OPEN, MASK_CLOSE, spacing=SPACING, ws=ws,
                                    stream=stream)
            else:
                L.lddmm_surface_distance(M0, M1, spacing=SPACING, ws=ws, stream=stream)
        e1.record(stream)
        torch.cuda.synchronize()
        avg_ms = e0.elapsed_time(e1) / MASK_CALLS
        per[name] = {"avg_us": 1e3 * avg_ms,
                     "GBs": MASK_ALG_BYTES[name] * n / (avg_ms * 1e-3) / 1e9}
    y_ms = ypass["ms"] / max(ypass["launches"], 1)
    y_achieved = MASK_XY_BYTES * n / (y_ms * 1e-3) / 1e9
    cpu = None
    if not args.no_cpu_baseline:
        log("cpu baseline (oracle) ...")
        cpu = masks_cpu_baseline(pair, masks_image(pair))
    d = d.cpu().numpy()
    out = {
        "metric": "mask voxels/s (target mask + two-sided surface distances)",
        "value": MASK_CALLS * args.steps * n / elapsed,
        "unit": "voxel/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": 1e3 * elapsed / args.steps,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "bit-packed masks, int32 squared distances, f64 distances",
        "data": "synthetic (seeded atlas-like image with grains and holes; atlas-like template mask)",
        "config": {"workload": "target mask (threshold, 50 um opening, 125 um closing) and "
                               "Hausdorff / median surface distances to the template mask, "
                               f"264x160x228 at 50 um; {MASK_CALLS} of each per step",
                   "grid": [264, 160, 228], "spacing_mm": SPACING, "tau": MASK_TAU,
                   "open_radius_mm": MASK_OPEN, "close_radius_mm": MASK_CLOSE},
        "roofline": {"bound": "hbm", "achieved": y_achieved, "peak": HBM_PEAK_GBS,
                     "unit": "GB/s", "frac": y_achieved / HBM_PEAK_GBS, "traffic": None,
                     "kernel": "k_edt_xy", "alg_bytes_per_voxel": MASK_XY_BYTES,
                     "avg_launch_ms": y_ms, "launches": ypass["launches"],
                     "voxels_per_launch": n},
        "calls": per,
        "distances_mm": {"hausdorff": float(d[0]), "median": float(d[1]),
                         "surface_voxels": [int(d[2]), int(d[3])]},
        "cpu_baseline": cpu,
    }
    print(json.dumps(out), flush=True)


def ctypes_grid(L, shape):
    import ctypes
    nz, ny, nx = shape
    return ctypes.byref(L._Grid(int(nx), int(ny), int(nz), float(SPACING)))


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=3)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--tune-only", action="store_true",
                    help="run the workload's autotuning (filling the tune cache) and exit, so "
                         "that profiled runs after it contain no trial launches")
    ap.add_argument("--trace-out", default=None)
    ap.add_argument("--workload", choices=("atlas", "atlas-rk4", "batched", "histmatch", "align",
                                           "masks"),
                    default="atlas",
                    help="atlas (default): the single-pair atlas registration; atlas-rk4: the "
                         "same with the paper's integrator (RK4, T=4); batched: 16 "
                         "uneven pairs in one grouped launch sequence vs 16 sequential runs; "
                         "histmatch: the Image-LDDMM histogram matching of the atlas pair; "
                         "align: rigid + affine pre-alignment of the atlas mask pair; "
                         "masks: target mask generation and surface distances")
    ap.add_argument("--summarize-profile", nargs=3, metavar=("DB", "OUT", "COMMAND"),
                    help="write a text summary of a rocprofv3 database and exit")
    ap.add_argument("--traffic-from", nargs=3, metavar=("FETCH_DB", "WRITE_DB", "OUT"),
                    help="compute calibrated per-launch sweep traffic from two counter runs and exit")
    args = ap.parse_args()
    if args.traffic_from:
        compute_traffic(*args.traffic_from)
        return
    if args.summarize_profile:
        summarize_profile(*args.summarize_profile)
        return
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (got --gpus {args.gpus}): a registration and "
              "its batched form each run on a single GPU", file=sys.stderr)
        sys.exit(2)
    if args.workload == "batched":
        bench_batched(args)
        return
    if args.workload == "histmatch":
        bench_histmatch(args)
        return
    if args.workload == "align":
        bench_align(args)
        return
    if args.workload == "masks":
        bench_masks(args)
        return
    if args.workload == "atlas-rk4":
        global T, FLAGS, INTEGRATOR
        T, INTEGRATOR = 4, "rk4"

    import torch
    from paper_1605_02060_amd import lddmm as L
    from paper_1605_02060_amd import synth

    L.load()
    assert torch.cuda.is_available(), "bench needs a GPU"
    if INTEGRATOR == "rk4":
        FLAGS = L.FLAG_RK4
    log("generating atlas-like pair ...")
    pair = synth.config_pair("atlas")
    dev = "cuda"
    tt = lambda a: torch.as_tensor(a, device=dev)
    M0, M1, MI0, MI1 = tt(pair.M0), tt(pair.M1), tt(pair.MI0), tt(pair.MI1)
    prm = L.Params(alpha=ALPHA, gamma=GAMMA, sigma=SIGMA, T=T, n_levels=LEVELS, iters=ITERS,
                   step=STEP, guard=GUARD, weight=(1.0, 0.0), flags=FLAGS)
    P = L.lddmm_comp_grid(pair.shape, prm, 0, SPACING)
    ws = L.workspace(pair.shape, prm, SPACING, dev)
    n_fine = P[0] * P[1] * P[2]
    attainable = attainable_bandwidth(torch, L)
    log(f"attainable bandwidth (library copy kernel): {attainable:.0f} GB/s")
    # launch shapes from the library's autotuner, outside the timed region
    from paper_1605_02060_amd import tune
    t_tune = time.perf_counter()
    choice = tune.autotune([{"M0": M0, "M1": M1, "MI0": MI0, "MI1": MI1, "spacing": SPACING}],
                           prm, verbose=False)
    tunables = {tune.NAMES[w]: v for w, v in choice.items()}
    log(f"autotune {time.perf_counter() - t_tune:.1f} s: {tunables}")
    if args.tune_only:
        return
    v = torch.zeros((T, 3) + P, dtype=torch.float32, device=dev)
    units = work_units(pair.shape)

    def step():
        v.zero_()
        return L.lddmm_register(M0, M1, MI0, MI1, params=prm, spacing=SPACING, v=v, ws=ws)

    # warmup; the first warmup step times every kernel class of the finest level, to
    # find the kernel with the largest total time and the K chain's time per step
    prof = None
    sweep_mask = sum(1 << L.PROF_CLASSES.index(c) for c in SWEEP_CLASSES)
    for w in range(max(args.warmup, 1)):
        if w == 0:
            L.lddmm_profile_begin(sweep_mask, n_fine)
        res = step()
        torch.cuda.synchronize()
        if w == 0:
            prof = L.lddmm_profile_end()
        log(f"warmup {w} done, status {res['status']}")
    # each class below is one kernel at the finest level (the edge classes hold the
    # first and last steps of a sweep, two kernels each, and are not candidates)
    dominant = max(ALG_BYTES, key=lambda k: prof[k]["ms"])
    cls_bit = 1 << L.PROF_CLASSES.index(dominant)

    # timed region: exactly K steps, HIP events around the dominant kernel
    L.lddmm_profile_begin(cls_bit, n_fine)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for k in range(args.steps):
        res = step()
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    live = L.lddmm_profile_end()[dominant]
    elapsed = t1 - t0
    ms_per_step = 1000.0 * elapsed / args.steps
    value = units * args.steps / elapsed

    tr = res["trace"].cpu().numpy()
    rej = int((tr[:, 6] == 0).sum())
    user_fine = int(np.prod(pair.shape))             # user voxels of the finest level
    avg_ms = live["ms"] / max(live["launches"], 1)
    vox_per_launch = live["voxels"] / max(live["launches"], 1)
    achieved = ALG_BYTES[dominant] * user_fine / (avg_ms * 1e-3) / 1e9
    achieved_padded = ALG_BYTES[dominant] * vox_per_launch / (avg_ms * 1e-3) / 1e9
    total_ms = sum(x["ms"] for x in prof.values())
    shares = {k: round(x["ms"] / total_ms, 4) for k, x in prof.items() if x["launches"]}
    per_launch_us = {k: round(1000.0 * x["ms"] / x["launches"], 2)
                     for k, x in prof.items() if x["launches"]}
    chain_ms = sum(prof[k]["ms"] / prof[k]["launches"] for k in K_CHAIN)
    chain_gbs = K_CHAIN_ALG_BYTES * user_fine / (chain_ms * 1e-3) / 1e9
    rk4 = FLAGS != 0

    out = {
        "metric": "voxel-timestep updates/s (flow+adjoint+K); time to target masked SSD",
        "value": value,
        "unit": "voxel-timestep/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_per_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic (seeded atlas-like template, sparse Poisson-labelled warped target)",
        "config": dict(workload_config(), tunables=tunables),
        "roofline": {"bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": achieved / HBM_PEAK_GBS,
                     "traffic": stored_traffic(dominant) if not rk4 else None,
                     "attainable": attainable, "frac_of_attainable": achieved / attainable,
                     "kernel": kernel_name(dominant, tunables, rk4),
                     "profile_class": dominant,
                     "alg_bytes_per_voxel": ALG_BYTES[dominant],
                     "voxels": "user voxels of the finest level (264x160x228); the kernel "
                               "runs on the padded 280x160x240 grid",
                     "user_voxels_per_launch": user_fine,
                     "padded_voxels_per_launch": vox_per_launch,
                     "achieved_on_padded_voxels": achieved_padded,
                     "frac_on_padded_voxels": achieved_padded / HBM_PEAK_GBS,
                     "measured_on": "finest-level launches of the timed steps (HIP events on the "
                                    "launch stream)",
                     "avg_launch_ms": avg_ms, "launches": live["launches"]},
        "k_chain": {"passes": list(K_CHAIN), "alg_bytes_per_voxel": K_CHAIN_ALG_BYTES,
                    "us_per_time_step": 1000.0 * chain_ms, "achieved_GBs": chain_gbs,
                    "frac": chain_gbs / HBM_PEAK_GBS,
                    "measured_on": "finest-level launches of the first warmup step"},
        "path_roofline": {"alg_bytes_per_voxel_timestep": B_ALG_PATH,
                          "achieved_GBs": value * B_ALG_PATH / 1e9,
                          "frac": value * B_ALG_PATH / 1e9 / HBM_PEAK_GBS},
        "finest_level_kernel_time_shares": shares,
        "finest_level_us_per_launch": per_launch_us,
        "level_final_E": [float(tr[i, 7]) for i in np.cumsum([it + 1 for it in ITERS]) - 1],
        "time_to_target_s": ms_per_step / 1000.0,
        "target_masked_ssd": last_accepted_D(tr),
        "rejected_slots": rej,
        "status": res["status"],
    }
    if args.trace_out:
        np.save(args.trace_out, tr)
    if not args.no_cpu_baseline:
        log("timing the oracle on a bounded sample ...")
        out["cpu_baseline"] = cpu_baseline(pair)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
