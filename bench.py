#!/usr/bin/env python3
"""Benchmark: batched adaptive-VQE steps at 14 qubits on one MI355X.

Workload: 64 independent states, each a 14-qubit register (7 spatial orbitals,
6 electrons, Jordan-Wigner) with its own seeded synthetic Hamiltonian
(2,596,863 CSR entries) and the shared 204-generator singles+doubles pool.
One step = one adaptive iteration for every state in one launch sequence:
H product with the FP64 energy reduction, the pool-gradient screen over all
204 generators, argmax selection, the fused fifth-order Taylor update and the
FP64 renormalisation.  Storage is FP32 (complex64, with an FP64 diagonal
shift); products and reductions are FP64.  Inputs are resident in HBM before
the timed region.  The throughput leg runs the K timed steps as one captured
graph of K steps (vqe_batch_run; each step takes its angles from the next row
of a device array), and reports beside it the same steps launched one graph
per step with a host-issued angle copy before each.

The headline leg's states are complex: each starts from a seeded complex state
of its particle sector, so the H product and the screen run in complex
arithmetic.  The Hamiltonians are held as their schedule's layout holds them
(value_form in the line: with the value dictionary, real magnitudes as codes
and, for a real H, the other entries' real parts).  Its algorithmic bytes count
the canonical CSR with complex values (int32 column + complex value per entry,
each vector once); the roofline counts the bytes of the stored form, which are
those that the kernel moves.
The real-value specialisation (real parts of a real H, real states from the
reference) is timed as a separate block with its own accounting.

Printed (one JSON line): Taylor-O(5) updates/s (each with its full screen),
the pool-gradient SpMV HBM GB/s, p50/p99 step latency over a dedicated
latency leg, the roofline of the dominant kernel (the H product), the mixed
10/12/14-qubit batch, the plain FP64 single-request GPU path, the serving
stream, and the FP64 oracle timed on the host cores.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0      # MI355X HBM3E peak
RUN_MAX = 1024             # steps per vqe_batch_run call (VQE_RUN_MAX_STEPS)


# state bytes that fit in LDS beside the staged row pointers (larger states are
# column-tiled)
LDS_STATE_BYTES = 147 * 1024
PMC_PROFILES = ("h_product_14q_64states_complex_pmc.md", "h_product_14q_64states_pmc.md",
                "h_product_16q_16states_pmc.md", "h_product_18q_16states_pmc.md",
                "h_product_20q_4states_pmc.md")


def _traffic_record(path: str, schedule: int, workload: str):
    import hashlib
    rec = {}
    with open(path) as f:
        for line in f:
            if ": " in line and not line.startswith((" ", "#", "|")):
                k, v = line.rstrip("\n").split(": ", 1)
                rec[k] = v
    try:
        if int(rec["schedule"]) != int(schedule) or rec.get("workload_key") != workload:
            return None
        h = hashlib.sha256()
        for src in rec["kernel_sources"].split():
            with open(os.path.join(ROOT, src), "rb") as f:
                h.update(f.read())
        if h.hexdigest() != rec["kernel_sources_sha256"]:
            return None
        return int(rec["traffic_bytes_per_launch"])
    except (KeyError, ValueError, OSError):
        return None


def measured_traffic(schedule: int, workload: str):
    """HBM bytes per H-product launch from a committed FETCH_SIZE/WRITE_SIZE
    profile of this workload and schedule (calibrated against a copy kernel of
    known size), or None when there is none or the kernel sources have changed
    since it was taken."""
    for name in PMC_PROFILES:
        path = os.path.join(ROOT, "profiles", name)
        if os.path.exists(path):
            t = _traffic_record(path, schedule, workload)
            if t is not None:
                return t
    return None


def vs_electrons() -> dict:
    import vqe_system as vs
    return vs.ELECTRONS


def plan_sched_x16(sched: int, ds) -> bool:
    """True when the batch plan reads 16-bit column codes for every state:
    the pipelined schedule asks for them and every state has at most 2^16
    rows (states larger than LDS take the column-tiled form with the codes)."""
    from paper_2606_29692_amd import binding as B
    return bool(sched & B.VQE_SPMV_X16) and bool(sched & B.VQE_SPMV_PREFETCH) and \
        bool(sched & B.VQE_SPMV_LDS) and all(d.H.dim <= 65536 for d in ds)


def plan_sched_real(sched: int, ds) -> bool:
    """True when the batch plan streams the real parts of every H (the codes
    are read, or the sliced layout of states that fit LDS, and every H is
    flagged real)."""
    from paper_2606_29692_amd import binding as B
    sliced = bool(sched & B.VQE_SPMV_SLICED) and not plan_tiled(ds)
    return (plan_sched_x16(sched, ds) or sliced) and bool(sched & B.VQE_SPMV_REAL) and \
        all(d.H.real for d in ds)


def plan_tiled(ds) -> bool:
    """True when some state is larger than the LDS state limit, so that the
    plan runs the column-tiled H product."""
    return any(d.H.dim * d.psi.element_size() > LDS_STATE_BYTES for d in ds)


def plan_sched_pad(sched: int, ds) -> bool:
    """True when the plan streams the complex values in the row-padded layout."""
    from paper_2606_29692_amd import binding as B
    return plan_sched_x16(sched, ds) and bool(sched & B.VQE_SPMV_PAD) and \
        not plan_sched_real(sched, ds)


BLK_ROWS, BLK_TILE_BYTES = 2048, 96 * 1024     # blocked layout of column-tiled states
SELLT_ROWS, SELLT_TILE_BYTES = 2048, 128 * 1024  # sliced layout of column-tiled states


def plan_sliced(sched: int, d) -> bool:
    """True when a state runs the sliced layout (one row per lane; column
    tiled, slab by slab, when the state is larger than LDS)."""
    from paper_2606_29692_amd import binding as B
    return bool(sched & B.VQE_SPMV_SLICED)


def plan_blocked(sched: int, d) -> bool:
    """True when a column-tiled state runs the blocked layout (every tiled
    state except the real-value form's, which keeps the CSR order)."""
    from paper_2606_29692_amd import binding as B
    big = d.H.dim * d.psi.element_size() > LDS_STATE_BYTES
    real_tiled = bool(sched & B.VQE_SPMV_REAL) and bool(sched & B.VQE_SPMV_X16) and d.H.real \
        and d.H.dim <= 65536
    return big and bool(sched & B.VQE_SPMV_LDS) and bool(sched & B.VQE_SPMV_PREFETCH) and \
        not real_tiled


def plan_dict(sched: int, d) -> bool:
    """True when a state's sliced layout keeps most values in a dictionary."""
    from paper_2606_29692_amd import binding as B
    return bool(sched & B.VQE_SPMV_VDICT) and bool(sched & B.VQE_SPMV_XIDX) and \
        d.psi.element_size() == 8 and d.H.dim <= 1 << 20


def stored_h_bytes(sched: int, ds, entries=None, layout_bytes=None) -> int:
    """Bytes the H-product kernel has to read and write per launch in the
    form it reads: row pointers, 2- or 4-byte columns, complex or real
    values (row-padded or not), the state and the result.  A blocked state
    reads each slab's row pointers once (per row block and column tile),
    16-bit tile-local codes and the complex values.  A sliced state reads its
    layout's entries (``entries``, from the plan; pads included) as 16-bit
    columns and complex values, 2 bytes of row order per row (per row and
    column tile when tiled) and 8 bytes per slice (and per slab); with the
    flip-mask indices, 4 bytes per three entries and at most 2 KiB of masks
    per row block in place of the columns.  With the value dictionary, the
    layout's device bytes (``layout_bytes``) without what only its build uses,
    and 10 KiB of tables per row block (8 KiB per row block and column tile)."""
    from paper_2606_29692_amd import binding as B
    x16, rv = plan_sched_x16(sched, ds), plan_sched_real(sched, ds)
    pad = rv or plan_sched_pad(sched, ds)
    tot = 0
    for i, d in enumerate(ds):
        if plan_dict(sched, d):
            build, tables = 4 * (5 * 1024 + d.H.dim) + 2 * d.H.dim, 10240 * -(-d.H.dim // BLK_ROWS)
            if d.H.dim * d.psi.element_size() > LDS_STATE_BYTES:
                slabs = d.H.dim // SELLT_ROWS * (d.H.dim * d.psi.element_size() // SELLT_TILE_BYTES)
                build = 26 * 4096 + d.H.dim // 8 + 6 * d.H.dim + 8 * 32 * slabs
                tables = 8192 * slabs
            tot += layout_bytes[i] - build + tables + 2 * d.H.dim * d.psi.element_size()
            continue
        if plan_sliced(sched, d):
            big = d.H.dim * d.psi.element_size() > LDS_STATE_BYTES
            nb = -(-d.H.dim // (SELLT_ROWS if big else BLK_ROWS))
            nt = -(-d.H.dim // (SELLT_TILE_BYTES // d.psi.element_size())) if big else 1
            vb = d.H.val.element_size() // (2 if rv else 1)
            xi = bool(sched & B.VQE_SPMV_XIDX) and not big
            codes = (entries[i] // 3 * 4 + 2048 * nb) if xi else 2 * entries[i]
            tot += 2 * d.H.dim * nt + 8 * nb * nt * (BLK_ROWS // 64 + (1 if big else 0)) + \
                codes + entries[i] * vb + 2 * d.H.dim * d.psi.element_size()
            continue
        if plan_blocked(sched, d):
            tc = BLK_TILE_BYTES // d.psi.element_size()
            nb, nt = -(-d.H.dim // BLK_ROWS), -(-d.H.dim // tc)
            tot += 4 * nb * nt * (BLK_ROWS + 1) + d.H.nnz * (2 + d.H.val.element_size()) + \
                2 * d.H.dim * d.psi.element_size()
            continue
        cb = 2 if x16 else 4
        vb = d.H.val.element_size() // (2 if rv else 1)
        nnz = d.H.nnz
        if pad and d.H.dim * d.psi.element_size() <= LDS_STATE_BYTES:
            # the padded layout: every row rounded up to a multiple of eight
            lens = np.diff(d.H.rowptr.cpu().numpy().astype(np.int64))
            nnz = int(((lens + 7) // 8 * 8).sum())
        tot += 4 * (d.H.dim + 1) + nnz * (cb + vb) + 2 * d.H.dim * d.psi.element_size()
    return tot


def log(msg: str):
    print(f"[bench] {msg}", file=sys.stderr, flush=True)


def percentile(a, q):
    return float(np.percentile(np.asarray(a), q))


def lat_stats(ms) -> dict:
    a = np.asarray(ms, dtype=np.float64)
    return {"p50_ms": percentile(a, 50), "p99_ms": percentile(a, 99),
            "p999_ms": percentile(a, 99.9), "mean_ms": float(a.mean()),
            "max_ms": float(a.max()), "n": int(a.size)}


def cpu_model() -> str:
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def cpu_baseline(system, psi0, reps: int, warm: int):
    """The FP64 oracle (test infrastructure, untuned) on one state of the
    benchmark workload (14 qubits, 6 electrons, JW, 204 generators; CSR built
    beforehand, untimed): medians over `reps` repetitions after `warm`
    warm-ups of the H product (sigma = H psi with the energy), the 204-generator
    screen (sigma reused), one Taylor-5 update and one whole adaptive step
    (energy, screen, selection, update, renormalisation), at one thread and at
    the process's thread count.  The headline rate is one whole step per
    update at the larger thread count."""
    from oracle import oracle as orc
    t_b = time.perf_counter()
    oH = orc.csr_from_pack(system.hamiltonian)
    pool = [orc.csr_from_pack(p) for p in system.pool]
    build_s = time.perf_counter() - t_b
    psi = np.asarray(psi0, dtype=np.complex128)
    _, _, _, sigma = orc.energy(oH, psi)
    k_sel, _ = orc.select(orc.gradients(pool, psi, sigma))
    theta = 0.05

    def step():
        e, _, _, sg = orc.energy(oH, psi)
        g = orc.gradients(pool, psi, sg)
        k, _ = orc.select(g)
        orc.normalize(orc.taylor5(pool[k], theta, psi))

    phases = {"h_spmv_energy": lambda: orc.energy(oH, psi),
              "pool_screen": lambda: orc.gradients(pool, psi, sigma),
              "taylor5": lambda: orc.taylor5(pool[k_sel], theta, psi),
              "adaptive_step": step}
    n_max = int(os.environ.get("OMP_NUM_THREADS", "0") or 0) or (os.cpu_count() or 1)
    t0 = time.perf_counter()
    per_threads = {}
    for nt in sorted({1, n_max}):
        orc.set_threads(nt)
        used = orc.threads()
        res = {}
        for name, fn in phases.items():
            for _ in range(warm):
                fn()
            ts = []
            for _ in range(reps):
                a = time.perf_counter()
                fn()
                ts.append(time.perf_counter() - a)
            res[name] = {"median_ms": float(np.median(ts)) * 1e3,
                         "min_ms": float(np.min(ts)) * 1e3}
        per_threads[str(used)] = res
    orc.set_threads(n_max)
    el = time.perf_counter() - t0
    top = per_threads[str(max(int(k) for k in per_threads))]
    return {"value": 1e3 / top["adaptive_step"]["median_ms"], "unit": "updates/s",
            "cores": max(int(k) for k in per_threads), "kind": "oracle",
            "sample": f"one 14-qubit state of the workload (2,596,863-entry H, 204 generators, "
                      f"complex start state), FP64; per phase the median of {reps} repetitions "
                      f"after {warm} warm-ups at 1 and {n_max} threads; {el:.1f} s of timing, "
                      f"CSR build {build_s:.2f} s untimed",
            "cpu_model": cpu_model(), "nproc": os.cpu_count(),
            "timer": "time.perf_counter (monotonic) around each oracle call",
            "phases_by_threads": per_threads,
            "paper_context": "the paper reports only memory for its CPU runs: 208.75 MB peak "
                             "resident set for the whole 14-qubit BeH2 pipeline on an Ubuntu "
                             "24.04 desktop (Sec. IV-C); no speed figure"}


def plain_fp64_path(ctx, system, n_req: int):
    """The plain FP64 single-request GPU path at 14 qubits: one request at a
    time, synchronised per request.  Returns (Taylor-only updates/s, full
    single-state adaptive steps/s, per-request latency statistics)."""
    import torch
    from paper_2606_29692_amd import batch as PB
    from paper_2606_29692_amd import binding as B
    ds = PB.device_system(ctx, system, "c128")
    sigma = torch.empty_like(ds.psi)
    A = ds.pool.ops[0]
    for _ in range(5):
        B.taylor5_apply(ctx, A, 0.01, ds.psi, renormalize=True)
    ctx.stream.synchronize()
    lat = []
    t0 = time.perf_counter()
    for i in range(n_req):
        a = time.perf_counter()
        B.taylor5_apply(ctx, ds.pool.ops[i % ds.pool.M], 0.01, ds.psi, renormalize=True)
        ctx.stream.synchronize()
        lat.append((time.perf_counter() - a) * 1e3)
    taylor_rate = n_req / (time.perf_counter() - t0)
    t0 = time.perf_counter()
    n_step = max(n_req // 2, 100)
    slat = []
    for i in range(n_step):
        a = time.perf_counter()
        B.energy(ctx, ds.H, ds.psi, sigma)
        g = B.pool_gradients(ctx, ds.H, ds.pool, ds.psi, sigma)
        k, _ = B.vqe_select(ctx, g)
        kk = int(k.cpu()[0])
        B.taylor5_apply(ctx, ds.pool.ops[kk], 0.01, ds.psi, renormalize=True)
        ctx.stream.synchronize()
        slat.append((time.perf_counter() - a) * 1e3)
    step_rate = n_step / (time.perf_counter() - t0)
    return taylor_rate, step_rate, lat_stats(lat), lat_stats(slat)


def serving_bench(n_requests: int, warm: int, log_fn=log, schedules: str = "tuned"):
    """Config C5: 64 resident runs with register sizes drawn from {8,...,16};
    Poisson request streams at 0.8x and 2x the capacity of the plain
    sequential FP64 single-request path; continuous batching (FP32 storage,
    slot groups per register size, one stream each) against that path.
    schedules: "default" (the library's per register size) or "tuned" (the
    autotuner's; sliced ones bind a layout built per run at admission)."""
    import torch
    import vqe_system as vs
    from paper_2606_29692_amd import binding as B
    from paper_2606_29692_amd import serve as S

    specs, _ = vs.config_c5(n_runs=64)
    systems = {r: vs.make_system(sp) for r, sp in enumerate(specs)}
    thetas = {r: vs.draw_thetas(sp.seed, 4096) for r, sp in enumerate(specs)}
    sizes = sorted({sp.n_qubits for sp in specs})
    ctx = B.Context(0, torch.cuda.Stream())
    # capacity of the sequential FP64 path: a burst served back to back
    burst = [S.Request(i, i % len(systems), 0.0) for i in range(256)]
    done = S.run_sequential(ctx, systems, burst, thetas)
    cap = len(done) / max(q.t_done for q in done)
    log_fn(f"serving: sequential FP64 capacity {cap:.0f} requests/s ({len(systems)} runs, "
           f"N in {sizes})")
    free, _ = torch.cuda.mem_get_info()
    budget = int(0.5 * free)
    out = {"runs": len(systems), "register_sizes": sizes, "requests": n_requests,
           "schedules": schedules,
           "warmup_requests": warm, "sequential_fp64_capacity_per_s": cap,
           "budget_bytes": budget}
    for factor in (0.8, 2.0):
        rate = factor * cap
        trace = S.poisson_trace(n_requests, rate, len(systems), seed=int(factor * 10))
        t_cold = time.perf_counter()
        ex = S.DeviceExecutor(systems, slots_per_group=16, dtype="c64",
                              schedules="tuned" if schedules == "tuned" else None)
        server = S.Server(ex, thetas, budget_bytes=budget)
        resident = server.prewarm()
        torch.cuda.synchronize()
        t_cold = time.perf_counter() - t_cold
        served = server.run_trace([S.Request(q.rid, q.run, q.t_arrival) for q in trace])
        cb = S.latency_summary(sorted(served, key=lambda q: q.rid), skip=warm)
        seq = S.run_sequential(ctx, systems, [S.Request(q.rid, q.run, q.t_arrival) for q in trace],
                               thetas)
        sq = S.latency_summary(sorted(seq, key=lambda q: q.rid), skip=warm)
        out[f"x{factor}"] = {"rate_per_s": rate, "continuous_batching": cb,
                             "sequential_fp64": sq, "evictions": server.evictions,
                             "failed": server.failed_count, "resident_runs": resident,
                             "cold_start_s": t_cold}
        log_fn(f"serving at {factor}x ({rate:.0f}/s): batched p50 {cb['p50_ms']:.3f} ms p99 "
               f"{cb['p99_ms']:.3f} ms p99.9 {cb['p999_ms']:.3f} ms {cb['updates_per_s']:.0f}/s "
               f"(n={cb['n']}); sequential p50 {sq['p50_ms']:.3f} ms p99 {sq['p99_ms']:.3f} ms")
        del ex, server
        torch.cuda.synchronize()
    ctx.close()
    return out


def timed_leg(plan, stream, n_states: int, thetas, K: int, W: int, L: int, R: int,
              tiled_screen: bool = False):
    """Time one batch plan's whole adaptive step (captured graphs):
      throughput  K steps between two events as ONE graph launch
                  (vqe_batch_run: step i takes its angles from row i of a
                  device array written before the timed region), after W
                  warm-up steps and one warm-up run; beside it the same K
                  steps as K whole-step graph launches with a host-issued
                  angle copy before each;
      latency     L steps with an event at every step boundary;
      H product   R back-to-back launches of the H products alone between two
                  events (the roofline's kernel duration: the events' own cost,
                  about 9 us each on this stack, is spread over the launches),
                  and R steps recording events before and after the H-product
                  graph and at the end (the product inside a step).
    thetas: device float64 [W + K + L + R + 1, n_states].  tiled_screen: the
    step flag for states known to be complex (the row-tiled screen)."""
    import torch
    Ev = lambda: torch.cuda.Event(enable_timing=True)   # noqa: E731
    t = 0

    def next_theta():
        nonlocal t
        plan.theta.copy_(thetas[t % thetas.shape[0]])
        t += 1

    ts = tiled_screen
    for _ in range(W):
        next_theta()
        plan.step(renorm=True, graph=True, tiled_screen=ts)
    ev3 = [Ev() for _ in range(3)]
    next_theta()
    plan.step_timed(ev3, renorm=True, graph=True, tiled_screen=ts)   # captures the split graphs
    # runs of at most RUN_MAX steps (the library's limit per call); the rows
    # of a later run are written on the plan's stream between the runs
    C = min(K, RUN_MAX)
    sizes = [C] * (K // C) + ([K % C] if K % C else [])
    rows = torch.empty((C, n_states), dtype=torch.float64, device=thetas.device)

    def fill_rows(n):
        nonlocal t
        idx = torch.arange(t, t + n, device=thetas.device) % thetas.shape[0]
        rows[:n].copy_(thetas[idx])
        t += n

    for n in sorted(set(sizes)):       # captures the graph of each run length
        fill_rows(n)
        plan.run(rows[:n], renorm=True, graph=True, tiled_screen=ts)
    fill_rows(sizes[0])
    torch.cuda.synchronize()
    start, stop = Ev(), Ev()
    start.record(stream)
    t_host = time.perf_counter()
    for i, n in enumerate(sizes):
        if i:
            fill_rows(n)
        plan.run(rows[:n], renorm=True, graph=True, tiled_screen=ts)
    stop.record(stream)
    torch.cuda.synchronize()
    wall = time.perf_counter() - t_host
    ms_per_step = start.elapsed_time(stop) / K
    start1, stop1 = Ev(), Ev()
    start1.record(stream)
    for _ in range(K):
        next_theta()
        plan.step(renorm=True, graph=True, tiled_screen=ts)
    stop1.record(stream)
    torch.cuda.synchronize()
    ms_single = start1.elapsed_time(stop1) / K
    bounds = [Ev() for _ in range(L + 1)]
    bounds[0].record(stream)
    for i in range(L):
        next_theta()
        plan.step(renorm=True, graph=True, tiled_screen=ts)
        bounds[i + 1].record(stream)
    torch.cuda.synchronize()
    step_lat = [bounds[i].elapsed_time(bounds[i + 1]) for i in range(L)]
    evs = [[Ev() for _ in range(3)] for _ in range(R)]
    for i in range(R):
        next_theta()
        plan.step_timed(evs[i], renorm=True, graph=True, tiled_screen=ts)
    torch.cuda.synchronize()
    h_ms = [e[0].elapsed_time(e[1]) for e in evs]
    rest_ms = [e[1].elapsed_time(e[2]) for e in evs]
    h_b2b = plan.time_products(R)
    return {"ms_per_step": ms_per_step, "updates_per_s": n_states * K / (ms_per_step * K / 1e3),
            "steps": K, "warmup": W, "host_wall_s": wall,
            "throughput_launch": f"the {K} steps as {len(sizes)} graph launch(es) of up to {C} "
                                 "steps (vqe_batch_run), angles row by row from a device array "
                                 "written before each run",
            "single_step_graphs": {"ms_per_step": ms_single,
                                   "updates_per_s": n_states / (ms_single / 1e3),
                                   "launch": "one whole-step graph per step, a host-issued angle "
                                             "copy before each"},
            "step_latency": lat_stats(step_lat),
            "h_product_ms": h_b2b, "h_product_launches_timed": R,
            "h_product_timing": "back-to-back launches of the H-product kernels between two HIP "
                                "events (vqe_batch_time_products)",
            "h_product_in_step_ms": float(np.mean(h_ms)),
            "h_product_in_step_ms_median": float(np.median(h_ms)),
            "rest_of_step_ms": float(np.mean(rest_ms))}


def eager_phases(plan, n: int = 10, tiled_screen: bool = False) -> dict:
    """Phase breakdown of the same step launched eagerly (7 events)."""
    import torch
    ev2 = [[torch.cuda.Event(enable_timing=True) for _ in range(7)] for _ in range(n)]
    for t in range(n):
        plan.step_timed(ev2[t], renorm=True, tiled_screen=tiled_screen)
    torch.cuda.synchronize()
    m = lambda a, b: float(np.mean([e[a].elapsed_time(e[b]) for e in ev2]))   # noqa: E731
    return {"h_spmv": m(0, 1), "screen": m(2, 3), "taylor": m(4, 5), "renorm": m(5, 6),
            "step": m(0, 6)}


def set_states(ds, systems, form: str):
    """Start every state from the reference (real) or from its seeded complex
    start state (FP32 storage rounds it)."""
    import torch
    import vqe_system as vs
    for d, s in zip(ds, systems):
        if form == "complex":
            d.psi.copy_(torch.from_numpy(vs.complex_start_state(s)).to(d.psi.dtype))
        else:
            d.reset()


def mixed_batch_leg(ctx, stream, pools_mf: bool, K: int, W: int, L: int, R: int):
    """Config C4: 64 states with N cycling over 10/12/14 (n_e 4/8/6), each with
    its own pool, one launch sequence per step, complex start states; the
    complex-value schedules chosen for the batch (each size's own, or one
    shared by all states when one H-product launch for the batch is faster)."""
    import torch
    import vqe_system as vs
    from paper_2606_29692_amd import batch as PB
    from paper_2606_29692_amd import tune as T
    specs, _ = vs.config_c4(n_states=64, mixed=True)
    systems = [vs.make_system(s) for s in specs]
    pools = PB.PoolCache(ctx, matrix_free=pools_mf)
    ds = [PB.device_system(ctx, s, "c64", pools) for s in systems]
    set_states(ds, systems, "complex")
    per_slot = T.schedules_for_batch(ctx, ds, value_form="complex")
    choice = T.last_batch_record(ctx, ds, value_form="complex")
    scheds = {d.n_qubits: s for d, s in zip(ds, per_slot)}
    plan = PB.make_batch(ctx, ds, schedules=per_slot)
    rng = np.random.default_rng(np.random.SeedSequence([4, 1]))
    th = torch.from_numpy(rng.uniform(-0.1, 0.1, size=(W + K + L + R + 1, len(ds)))).to("cuda")
    leg = timed_leg(plan, stream, len(ds), th, K, W, L, R, tiled_screen=pools_mf)
    nb = PB.bytes_per_step(ds)
    plan.close()
    by_n = {str(n): sum(1 for d in ds if d.n_qubits == n) for n in scheds}
    out = {"workload": "64 states, N = (10, 12, 14)[i mod 3] (22/21/21), n_e 4/8/6, JW, own "
                       "pool per size (54/92/204), complex start states, FP32 storage",
           "states_by_qubits": by_n, "schedules": {str(k): v for k, v in sorted(scheds.items())},
           "schedule_choice": {"shared": choice["shared"], "own_per_size": choice["own"],
                               "h_product_ms_by_choice": choice["ms"]} if choice else None,
           "algorithmic_bytes_per_step": nb,
           "h_product_GBps": nb["h_spmv"] / (leg["h_product_ms"] / 1e3) / 1e9, **leg}
    del ds, pools
    return out


def main():
    ap = argparse.ArgumentParser(description=__doc__.split("\n")[0])
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=100)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--latency-steps", type=int, default=200,
                    help="steps of the latency leg (an event at every step boundary)")
    ap.add_argument("--h-timed-steps", type=int, default=100,
                    help="steps whose H-product graph is bracketed by events (roofline)")
    ap.add_argument("--states", type=int, default=64)
    ap.add_argument("--dtype", choices=["c64", "c128"], default="c64")
    ap.add_argument("--value-form", choices=["complex", "real"], default="complex",
                    help="headline leg: interleaved complex values and complex states (the "
                         "contract), or the real-value specialisation")
    ap.add_argument("--real-block", action=argparse.BooleanOptionalAction, default=True,
                    help="also time the real-value specialisation as a separate block")
    ap.add_argument("--schedule", type=int, default=0,
                    help="H product schedule of the headline leg (0: tuned)")
    ap.add_argument("--cpu-reps", type=int, default=20)
    ap.add_argument("--cpu-warmup", type=int, default=3)
    ap.add_argument("--matrix-free", action=argparse.BooleanOptionalAction, default=True,
                    help="screen and update from the generators' matrix-free records "
                         "(no pool CSR) instead of the pool's pair tables")
    ap.add_argument("--line-search-steps", type=int, default=20,
                    help="also time this many steps with the angle chosen by line search (0: skip)")
    ap.add_argument("--adapt-steps", type=int, default=12,
                    help="also run this many adaptive steps from the reference with line "
                         "search, without and with re-optimisation of every angle (0: skip)")
    ap.add_argument("--mixed-batch", action=argparse.BooleanOptionalAction, default=True,
                    help="also time the mixed 10/12/14-qubit 64-state batch")
    ap.add_argument("--qubits", type=int, default=14, choices=sorted(vs_electrons()),
                    help="register size of every state (the headline workload is 14)")
    ap.add_argument("--mapping", choices=["jw", "bk"], default="jw")
    ap.add_argument("--pool-order", choices=["canonical", "family"], default="canonical",
                    help="pool order: canonical, or grouped by commuting family (Alg. 1)")
    ap.add_argument("--retune", action="store_true",
                    help="time every H product schedule even when a tuned one is cached")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-plain", action="store_true")
    ap.add_argument("--serve-requests", type=int, default=4096,
                    help="requests per serving point (0: skip the serving measurement)")
    ap.add_argument("--serve-warmup", type=int, default=256)
    ap.add_argument("--serve-schedules", choices=["default", "tuned"], default="tuned",
                    help="H product schedules of the serving executor: the autotuner's per "
                         "register size (sliced ones bind a layout built once per run), or the "
                         "library's defaults")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (asked for --gpus {args.gpus}): states are "
              "independent, so a multi-GPU run would place whole states per GPU; no figure "
              "at several GPUs is produced", file=sys.stderr)
        sys.exit(2)

    import torch
    import vqe_system as vs
    from paper_2606_29692_amd import batch as PB
    from paper_2606_29692_amd import binding as B
    from paper_2606_29692_amd import tune as T

    stream = torch.cuda.Stream()           # default priority
    torch.cuda.set_stream(stream)
    ctx = B.Context(0, stream)
    n_cu, devname = ctx.info()
    log(f"device {devname}, {n_cu} CUs")

    if args.qubits == 14 and args.mapping == "jw":
        specs, _ = vs.config_c4(n_states=args.states, mixed=False)
    else:
        # the same seeds as the 14-qubit workload, at another size or mapping
        specs = [vs.SystemSpec(args.qubits, vs.ELECTRONS[args.qubits], args.mapping, False,
                               vs.system_seed(44, i)) for i in range(args.states)]
    t0 = time.perf_counter()
    systems = [vs.make_system(s) for s in specs]
    # commuting-family partition of the pool (Alg. 1): graph on the device,
    # greedy colouring on the host; optionally reorder the pool so that
    # families are contiguous
    mfp = B.MfPool(systems[0].pool)
    g0 = time.perf_counter()
    adj = B.noncommutation_graph(ctx, mfp)
    fam = B.partition_greedy(adj)
    partition = {"generators": int(mfp.M), "noncommuting_pairs": int(adj.sum()) // 2,
                 "families": int(fam.max()) + 1,
                 "graph_and_colouring_ms": (time.perf_counter() - g0) * 1e3,
                 "pool_order": args.pool_order}
    mfp.close()
    log(f"partition: {partition['families']} commuting families of {partition['generators']} "
        f"generators ({partition['noncommuting_pairs']} non-commuting pairs), "
        f"{partition['graph_and_colouring_ms']:.1f} ms")
    if args.pool_order == "family":
        perm = np.argsort(fam, kind="stable")
        for s in systems:
            s.pool = [s.pool[j] for j in perm]
    pools = PB.PoolCache(ctx, matrix_free=args.matrix_free)
    ds = [PB.device_system(ctx, s, args.dtype, pools) for s in systems]
    torch.cuda.synchronize()
    log(f"setup: {len(ds)} systems built on the device in {time.perf_counter() - t0:.1f} s")
    K, W, L, R = args.steps, args.warmup, args.latency_steps, args.h_timed_steps
    rng = np.random.default_rng(np.random.SeedSequence([44, 1]))
    thetas = torch.from_numpy(rng.uniform(-0.1, 0.1, size=(W + K + L + R + 1, len(ds)))).to("cuda")
    wl = f"{len(ds)}x{args.qubits}q-{args.mapping}-{args.dtype}"

    def run_form(form: str, sched_given: int = 0):
        """Tune (or take) the schedule for a value form, set the states, and
        time the leg; returns (schedule, leg record, eager phases, plan)."""
        vf = "complex" if form == "complex" else "any"
        sched = sched_given or T.schedule_for(ctx, ds[0], systems=ds, retune=args.retune,
                                              value_form=vf)
        if T._last_timings:
            log(f"tuner ({form}; ms of the batched H product): " +
                ", ".join(f"{k}: {v:.3f}" for k, v in sorted(T._last_timings.items())))
            T._last_timings.clear()
        set_states(ds, systems, form)
        plan = PB.make_batch(ctx, ds, schedules=[sched] * len(ds))
        # complex states take the row-tiled screen (the step flag for them)
        ts = form == "complex" and args.matrix_free
        leg = timed_leg(plan, stream, len(ds), thetas, K, W, L, R, tiled_screen=ts)
        leg["layout_entries"] = [plan.layout_entries(i) for i in range(len(ds))]
        leg["layout_bytes"] = None
        if plan_dict(sched, ds[0]):
            leg["layout_bytes"] = []
            for d in ds:
                lay = B.Layout(ctx, d.H, sched)
                leg["layout_bytes"].append(lay.nbytes())
                lay.close()
        ph = eager_phases(plan, tiled_screen=ts)
        leg["tiled_screen"] = ts
        return sched, leg, ph, plan

    def form_record(form: str, sched: int, leg: dict, ph: dict) -> dict:
        acc = "complex" if form == "complex" else "real"
        nb = PB.bytes_per_step(ds, value_form=acc)
        stored = stored_h_bytes(sched, ds, leg.pop("layout_entries"), leg.pop("layout_bytes"))
        dic = plan_dict(sched, ds[0])
        h_s = leg["h_product_ms"] / 1e3
        achieved = nb["h_spmv"] / h_s / 1e9
        x16, rv = plan_sched_x16(sched, ds), plan_sched_real(sched, ds)
        return {
            "schedule": sched,
            "value_form": "dictionary of real magnitudes, other entries " +
                          ("their real parts" if ds[0].H.real else "complex") if dic else
                          "real parts" if rv else "complex",
            "state_form": form, "algorithmic_bytes_per_step": nb,
            "byte_accounting": ("canonical CSR: int32 column + complex value per entry, each "
                                "vector once" if acc == "complex" else
                                "canonical CSR with real values (half the complex element) "
                                "for a real H: the specialisation's own accounting, not the "
                                "contract's") +
                               ("; the kernel reads the smaller stored form (stored_bytes_per_"
                                "launch at stored_GBps, the roofline's figures), so the canonical "
                                "bytes' rate (h_product_GBps) is no HBM rate and may pass the peak"),
            "h_product_GBps": achieved, "h_product_frac_of_peak": achieved / HBM_PEAK_GBS,
            "traffic_bytes_per_launch": measured_traffic(sched, wl),
            "stored_bytes_per_launch": stored, "stored_GBps": stored / h_s / 1e9,
            "column_form": ((("16-bit" if plan_tiled(ds) else "12-bit") + " codes of (flip mask, "
                             "magnitude) pairs and the sign, and for the other entries " if dic else "") +
                            ("10-bit flip-mask indices (three per 32-bit word)"
                             if sched & B.VQE_SPMV_XIDX and not plan_tiled(ds) else "16-bit columns") +
                            ", one row per lane in slices of 64 rows sorted by "
                            "length" + (" per column tile" if plan_tiled(ds) else "") +
                            (", real values" if rv else "")
                            if all(plan_sliced(sched, d) for d in ds) else
                            ("16-bit col^row codes" if x16 else "int32 CSR columns") +
                            (", rows padded to groups of eight" if rv or plan_sched_pad(sched, ds)
                             else "")),
            "pool_gradient_spmv_GBps": (nb["h_spmv"] + nb["pool_screen"]) /
                                       ((leg["h_product_ms"] + ph["screen"]) / 1e3) / 1e9,
            "eager_phase_ms": ph, **leg}

    form = args.value_form
    sched, leg, ph, plan = run_form(form, args.schedule)
    head = form_record(form, sched, leg, ph)
    nbytes = head["algorithmic_bytes_per_step"]
    log(f"{form} form (schedule {sched}): {leg['ms_per_step']:.3f} ms/step = "
        f"{leg['updates_per_s']:.0f} updates/s (graphs of up to {RUN_MAX} steps; one graph per "
        f"step: {leg['single_step_graphs']['ms_per_step']:.3f} ms/step); step latency p50 "
        f"{leg['step_latency']['p50_ms']:.3f} p99 {leg['step_latency']['p99_ms']:.3f} ms "
        f"(n={leg['step_latency']['n']}); H product {leg['h_product_ms'] * 1e3:.1f} us "
        f"({head['stored_GBps']:.0f} GB/s stored, frac {head['stored_GBps'] / HBM_PEAK_GBS:.3f}; "
        f"{head['h_product_GBps']:.0f} GB/s of canonical CSR bytes); eager "
        f"screen {ph['screen'] * 1e3:.1f} us, Taylor {ph['taylor'] * 1e3:.1f} us, renorm "
        f"{ph['renorm'] * 1e3:.1f} us")
    plan.close()

    real_block = None
    if args.real_block and form == "complex" and all(d.H.real for d in ds):
        rs, rleg, rph, rplan = run_form("real")
        real_block = form_record("real", rs, rleg, rph)
        real_block["note"] = ("real-value specialisation: the real parts of a real H streamed "
                              "in a row-padded layout, real states from the reference screened "
                              "and multiplied in real arithmetic; reported apart from the "
                              "complex contract")
        log(f"real-value form (schedule {rs}): {rleg['ms_per_step']:.3f} ms/step = "
            f"{rleg['updates_per_s']:.0f} updates/s; H product {rleg['h_product_ms'] * 1e3:.1f} us")
    else:
        rplan = None

    # the same step with the angle chosen by line search (two more H products
    # per state); a separate figure, not the headline value.  Runs on the
    # real-value plan (states from the reference) when there is one.
    lplan = rplan if rplan is not None else PB.make_batch(ctx, ds, schedules=[sched] * len(ds))
    line_search = None
    if args.line_search_steps > 0:
        lplan.set_line_search(1.0)
        for _ in range(2):
            lplan.step(renorm=True, graph=True, line_search=True)
        torch.cuda.synchronize()
        e_before = lplan.energies.view(-1, 3)[:, 0].clone()
        l0, l1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        l0.record(stream)
        for _ in range(args.line_search_steps):
            lplan.step(renorm=True, graph=True, line_search=True)
        l1.record(stream)
        torch.cuda.synchronize()
        ls_ms = l0.elapsed_time(l1) / args.line_search_steps
        lplan.step(update=False)
        torch.cuda.synchronize()
        drop = float((e_before - lplan.energies.view(-1, 3)[:, 0]).mean())
        lplan.set_line_search(0.0)
        line_search = {"ms_per_step": ls_ms, "updates_per_s": len(ds) / (ls_ms / 1e3),
                       "steps": args.line_search_steps, "theta_max": 1.0,
                       "mean_energy_drop_Ha": drop}
        log(f"line search: {ls_ms:.3f} ms/step ({len(ds) / (ls_ms / 1e3):.0f} updates/s), "
            f"mean energy drop over {args.line_search_steps} steps {drop:.4f} Ha")

    # adaptive runs from the reference: the angle of each new update by line
    # search, then optionally one sweep re-optimising every angle (cyclic
    # coordinate line search); separate figures, not the headline value
    adapt = None
    if args.adapt_steps > 0:
        S, eps = args.adapt_steps, 1e-3
        adapt = {"steps": S, "epsilon": eps, "theta_max": 1.0}
        for mode in ("line_search", "line_search+reoptimization"):
            for d in ds:
                d.reset()
            lplan.set_line_search(1.0)
            hist = PB.AnsatzHistory(lplan, S)
            gm = torch.zeros((S, len(ds)), dtype=torch.float64, device="cuda")
            en = torch.zeros((S + 1, len(ds)), dtype=torch.float64, device="cuda")
            r_ms = 0.0
            torch.cuda.synchronize()
            a0, a1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a0.record(stream)
            for t in range(S):
                lplan.step(renorm=True, line_search=True)
                gm[t].copy_(lplan.gmax)
                en[t].copy_(lplan.energies.view(-1, 3)[:, 0])
                hist.record()
                if mode != "line_search":
                    r0, r1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                    r0.record(stream)
                    hist.reoptimize(1, 1.0)
                    r1.record(stream)
                    r1.synchronize()
                    r_ms += r0.elapsed_time(r1)
            a1.record(stream)
            lplan.step(update=False)
            en[S].copy_(lplan.energies.view(-1, 3)[:, 0])
            torch.cuda.synchronize()
            total = a0.elapsed_time(a1)
            g = gm.cpu().numpy()
            e = en.cpu().numpy()
            below = g < eps
            conv = [int(np.argmax(below[:, i])) if below[:, i].any() else None
                    for i in range(len(ds))]
            adapt[mode] = {"ms_total": total, "reoptimization_ms_total": r_ms if r_ms else None,
                           "mean_energy_drop_Ha": float((e[0] - e[S]).mean()),
                           "mean_final_gmax": float(np.abs(lplan.gmax.cpu().numpy()).mean()),
                           "states_converged": int(sum(c is not None for c in conv))}
            log(f"adaptive run ({mode}): {S} steps in {total:.1f} ms, mean energy drop "
                f"{(e[0] - e[S]).mean():.4f} Ha, mean final max|g| "
                f"{adapt[mode]['mean_final_gmax']:.2e}, {adapt[mode]['states_converged']} of "
                f"{len(ds)} states reached max|g| < {eps:g}")
        lplan.set_line_search(0.0)
    lplan.close()

    mixed = None
    if args.mixed_batch and args.qubits == 14 and args.dtype == "c64":
        mixed = mixed_batch_leg(ctx, stream, args.matrix_free, K, W, L, R)
        log(f"mixed 10/12/14 batch: {mixed['ms_per_step']:.3f} ms/step = "
            f"{mixed['updates_per_s']:.0f} updates/s, H product {mixed['h_product_ms'] * 1e3:.1f} us "
            f"({mixed['h_product_GBps']:.0f} GB/s), step p99 {mixed['step_latency']['p99_ms']:.3f} ms; "
            f"schedules {mixed['schedules']}")

    # practical HBM ceiling for context: a plain device copy (read + write) of 2 GiB
    # (an elementwise kernel, dst = src * 1, so profilers see it as a kernel)
    src = torch.ones(1 << 28, dtype=torch.float64, device="cuda")
    dst = torch.empty_like(src)
    torch.mul(src, 1.0, out=dst)
    torch.cuda.synchronize()
    c0, c1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    c0.record(stream)
    for _ in range(5):
        torch.mul(src, 1.0, out=dst)
    c1.record(stream)
    torch.cuda.synchronize()
    copy_gbs = 5 * 2 * src.numel() * 8 / (c0.elapsed_time(c1) / 1e3) / 1e9
    s0, s1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    acc = src.sum()
    s0.record(stream)
    for _ in range(5):
        acc = src.sum()
    s1.record(stream)
    torch.cuda.synchronize()
    read_gbs = 5 * src.numel() * 8 / (s0.elapsed_time(s1) / 1e3) / 1e9
    del src, dst, acc
    log(f"device copy: {copy_gbs:.0f} GB/s (read + write); device sum: {read_gbs:.0f} GB/s (read)")

    plain = None
    if not args.no_plain:
        tr, sr, tlat, slat = plain_fp64_path(ctx, systems[0], 200)
        plain = {"taylor_updates_per_s": tr, "adaptive_steps_per_s": sr,
                 "taylor_request_latency": tlat, "step_request_latency": slat,
                 "batched_speedup_updates": head["updates_per_s"] / tr}
        log(f"plain FP64 single-request path: {tr:.0f} Taylor updates/s "
            f"(p50 {tlat['p50_ms'] * 1e3:.0f} us), {sr:.0f} steps/s (p50 "
            f"{slat['p50_ms']:.3f} ms)")

    cpu = None
    if not args.no_cpu_baseline and args.qubits == 14:
        psi0 = vs.complex_start_state(systems[0]).astype(np.complex64).astype(np.complex128)
        cpu = cpu_baseline(systems[0], psi0, args.cpu_reps, args.cpu_warmup)
        ph1 = cpu["phases_by_threads"]
        log(f"cpu baseline ({cpu['cpu_model']}): {cpu['value']:.1f} updates/s on {cpu['cores']} "
            f"threads; medians " + "; ".join(
                f"{nt} thr: " + ", ".join(f"{k} {v['median_ms']:.2f} ms" for k, v in r.items())
                for nt, r in ph1.items()))

    serving = None
    if args.serve_requests > 0:
        serving = serving_bench(args.serve_requests, min(args.serve_warmup,
                                                         args.serve_requests // 4),
                                schedules=args.serve_schedules)

    hnnz = ds[0].H.nnz
    tiled = plan_tiled(ds)
    out = {
        "metric": f"Taylor-O(5) updates/s + pool-gradient SpMV HBM GB/s at {args.qubits} qubits; "
                  f"p99 latency",
        "value": head["updates_per_s"],
        "unit": "updates/s",
        "n_gpus": 1,
        "steps": K,
        "warmup": W,
        "ms_per_step": head["ms_per_step"],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32" if args.dtype == "c64" else "f64",
        "accumulate": "f64",
        "data": "synthetic (seeded molecule-shaped random integrals; seeded complex start "
                "states in each state's particle sector; no molecular data)",
        "config": {
            "workload": f"{len(ds)} independent states x {args.qubits} qubits ({args.qubits // 2} "
                        f"orbitals, {vs.ELECTRONS[args.qubits]} electrons, {args.mapping.upper()}), "
                        f"H nnz {hnnz} each, pool {ds[0].pool.M} shared; one adaptive step per state per "
                        f"launch sequence (H SpMV + FP64 energy, {ds[0].pool.M}-generator gradient screen, "
                        f"argmax, fused Taylor-O(5), FP64 renorm); values: {head['value_form']}; "
                        f"{form} states",
            "states": len(ds), "n_qubits": args.qubits, "n_electrons": vs.ELECTRONS[args.qubits],
            "mapping": args.mapping, "pool": ds[0].pool.M, "storage": args.dtype,
            "value_form": head["value_form"], "state_form": form,
            "spmv_schedule": sched,
            "pool_form": "matrix-free records" if args.matrix_free else "pair tables from the pool CSR",
        },
        "pool_gradient_spmv_GBps": head["pool_gradient_spmv_GBps"],
        "p50_step_ms": head["step_latency"]["p50_ms"],
        "p99_step_ms": head["step_latency"]["p99_ms"],
        "step_latency": head["step_latency"],
        "eager_phase_ms": head["eager_phase_ms"],
        "algorithmic_bytes_per_step": nbytes,
        # the bytes that the kernel has to move, in the form it reads
        "roofline": {"bound": "hbm", "achieved": head["stored_GBps"], "peak": HBM_PEAK_GBS,
                     "unit": "GB/s", "frac": head["stored_GBps"] / HBM_PEAK_GBS,
                     "traffic": measured_traffic(sched, wl),
                     "traffic_unit": "bytes per launch (HBM read + write, PMC-calibrated)",
                     "kernel": (f"sliced column-tiled H product of all {len(ds)} states "
                                f"(k_spmv_sellt: row blocks of {SELLT_ROWS}, column tiles of "
                                f"{SELLT_TILE_BYTES // 1024} KiB, one row per lane, accumulators in LDS)"
                                if tiled and all(plan_sliced(sched, d) for d in ds) else
                                f"blocked column-tiled H product of all {len(ds)} states "
                                f"(k_spmv_blk: row blocks of {BLK_ROWS}, column tiles of "
                                f"{BLK_TILE_BYTES // 1024} KiB, accumulators in LDS)"
                                if tiled and all(plan_blocked(sched, d) for d in ds) else
                                f"column-tiled H product of all {len(ds)} states (k_spmv_tiled, "
                                f"then k_spmv_tile_sum)" if tiled else
                                f"H product of all {len(ds)} states (one launch of the schedule's "
                                f"kernel: k_spmv_sell, k_spmv_lds_pf, k_spmv_lds or k_spmv_energy)"),
                     "bytes_per_launch": head["stored_bytes_per_launch"],
                     "launch_ms": head["h_product_ms"],
                     "launches_timed": head["h_product_launches_timed"],
                     "canonical_csr_bytes_per_launch": nbytes["h_spmv"],
                     "canonical_csr_GBps": head["h_product_GBps"],
                     "column_form": head["column_form"],
                     "value_form": head["value_form"]},
        "headline_leg": head,
        "real_value_form": real_block,
        "mixed_batch_c4": mixed,
        "plain_fp64_single_request": plain,
        "line_search": line_search,
        "adaptive_runs": adapt,
        "partition": partition,
        "serving": serving,
        "p99_latency_ms": (serving["x0.8"]["continuous_batching"]["p99_ms"] if serving
                           else None),
        "device_copy_GBps": copy_gbs,
        "device_read_GBps": read_gbs,
        "cpu_baseline": cpu,
        "host_wall_s": head["host_wall_s"],
    }
    print(json.dumps(out), flush=True)
    ctx.close()


if __name__ == "__main__":
    main()
