"""Throughput of list-mode MLEM reconstruction on one MI355X.

Workload (default ``prod400``): two strips at y = +-450 mm of length 500 mm, a 400 x 400 grid of
2 mm pixels, resolution sigma_z = 10 mm and sigma_dl = 63 mm, 10M synthetic events drawn from the
Appendix A phantom with four hot disks, sensitivity image computed once.  One step is one full
10-iteration reconstruction from rho^0 = 1 (where s > 0) of all 10M events, with the events
already in HBM and the per-event preparation done once before the timed region.

Prints one JSON line: events x iterations per second, the roofline of the dominant kernel (the
MLEM event pass, timed with HIP events on its own stream inside the timed region) and the
single-threaded double-precision oracle timed on a bounded sample of the same workload.
"""

from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

# (event, in-ellipse pixel) pairs per second of the event pass's own arithmetic with nothing beside it: the
# exponent's polynomial along the row (6 FMAs or multiplications for the two pixels at +-x), v_exp_f32, m = P rho
# and D += m, the back-projection's scale, whose bits are the fixed-point addend.  Measured by the microbenchmark
# (profiles/microbench_rates.md): the classes of VALU instructions run at rates of their own, from 19e12
# lanes a second (v_exp_f32) to 64e12 (v_add_f32), so no count of issue slots bounds a mix of them.
PEAK_PAIRS = 5.36e12
# HBM bytes per event pass, from rocprofv3 FETCH_SIZE and WRITE_SIZE counters scaled by what the same
# counters read for a 256 MiB device copy, keyed by the hash of the kernel sources they were taken
# on and the plan code (reported only while both are unchanged).
MEASURED_TRAFFIC = {"2331c9061ba0aa49:2205": 4005022421}


def kernel_source_hash() -> str:
    """sha256 prefix of the kernel sources (paper_1502_07478_amd/csrc/*, sorted by name) with their
    comments and blank lines removed, so that the figure follows the code, not its prose."""
    import glob
    import hashlib
    import re
    h = hashlib.sha256()
    for f in sorted(glob.glob(os.path.join(ROOT, "paper_1502_07478_amd", "csrc", "*"))):
        with open(f, encoding="utf-8") as fh:
            text = fh.read()
        text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
        text = re.sub(r"//[^\n]*", "", text)
        lines = [ln.rstrip() for ln in text.splitlines()]
        h.update("\n".join(ln for ln in lines if ln).encode())
    return h.hexdigest()[:16]


# Floating-point operations per pair of the kernel evaluation, forward sum and back-projection: 8.5
# FLOP (FMA = 2) and the transcendental counted as one; priced against the published FP32 vector peak
# of the MI355X (157.3 TFLOP/s, which counts packed FP32)
FLOPS_PER_PAIR = 9.5
PEAK_FP32_TFLOPS = 157.3


def host_cpu_model() -> str:
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    import platform
    return platform.processor() or "unknown"


def _events_of(w):
    return w.events(workers=1)


def measure_batched(jpet, torch, gen_workers=16):
    """64 independent reconstructions (grids 128/256/512, sigma_z 8..15, sigma_dl 40..90 mm,
    50k..2M events), 10 iterations each: one batched call against the instances run one after
    another with jpet_mlem_iterate (both with prepared workspaces)."""
    import multiprocessing as mp

    from jpet_synth.configs import batch_instances
    base = batch_instances()
    if gen_workers > 1:
        with mp.get_context("spawn").Pool(gen_workers) as pool:
            evs = pool.map(_events_of, base)
    else:
        evs = [_events_of(w) for w in base]
    n_iter = base[0].n_iter
    inst, rho0 = [], []
    for w, e in zip(base, evs):
        g = jpet.geometry(**w.geometry())
        s = jpet.sensitivity(g)
        r0 = (s > 0).to(torch.float32)
        inst.append((g, torch.from_numpy(e).cuda(), s, r0.clone()))
        rho0.append(r0)
    total = sum(len(e) for e in evs)
    # plain: one instance after another
    plain_ws = []
    for g, ev, s, rho in inst:
        ws = jpet.workspace(g, ev.shape[0])
        jpet.prepare(g, ev, ws)
        plain_ws.append(ws)
    for (g, ev, s, rho), r0, ws in zip(inst, rho0, plain_ws):  # warm-up
        rho.copy_(r0)
        jpet.mlem_iterate(g, ev, rho, 1, s=s, ws=ws, prepared=True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for (g, ev, s, rho), r0, ws in zip(inst, rho0, plain_ws):
        rho.copy_(r0)
        jpet.mlem_iterate(g, ev, rho, n_iter, s=s, ws=ws, prepared=True)
    torch.cuda.synchronize()
    t_plain = time.perf_counter() - t0
    del plain_ws
    torch.cuda.empty_cache()
    t0 = time.perf_counter()
    b = jpet.BatchedMLEM(inst, tuned=True)
    torch.cuda.synchronize()
    setup_s = time.perf_counter() - t0
    st = b.iterate(0, want_stats=True)
    pairs = sum(x["n_pairs"] for x in st)
    b.run(n_iter)  # captures the graph of n_iter iterations; the first launch warms up
    torch.cuda.synchronize()
    times = []
    for _ in range(3):
        for (g, ev, s, rho), r0 in zip(inst, rho0):
            rho.copy_(r0)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        b.run(n_iter)  # one graph launch: n_iter iterations of all 64 instances
        torch.cuda.synchronize()
        times.append(time.perf_counter() - t0)
    t_batched = sorted(times)[1]
    return {"instances": len(base), "events": total, "iterations": n_iter, "pairs_per_iteration": pairs,
            "plain_s": round(t_plain, 4), "batched_s": round(t_batched, 4),
            "speedup": round(t_plain / t_batched, 3), "batched_setup_s": round(setup_s, 2),
            "batched_events_iterations_per_s": round(total * n_iter / t_batched, 1),
            "batched_pairs_per_s": round(pairs * n_iter / t_batched, 1)}


def measure_gradient(jpet, torch, gen_workers=None):
    """Log-likelihood with its image and resolution gradients on 1M events at 200x200 px of 2.5 mm
    (events/s), against plain MLEM on the same events (events x iterations / s)."""
    from jpet_synth import get_workload
    from paper_1502_07478_amd import tune
    w = get_workload("grad200")
    ev = torch.from_numpy(w.events(workers=gen_workers)).cuda()
    g0 = jpet.geometry(**w.geometry())
    g = tune.tuned(g0, ev)  # the MLEM pass's tuned plan
    s = jpet.sensitivity(g)
    rho = (s > 0).to(torch.float32)
    ws = jpet.workspace(g, ev.shape[0])
    jpet.prepare(g, ev, ws)
    n_pairs = jpet.mlem_iterate(g, ev, rho, 0, s=s, ws=ws, prepared=True, want_stats=True)["n_pairs"]
    jpet.mlem_iterate(g, ev, rho, 5, s=s, ws=ws, prepared=True)
    reps = 5
    gl = jpet.with_plan(g0, tune.loglik_plan_for(g0, ev, rho, s))  # the log-likelihood pass's tuned plan
    wsl = jpet.loglik_workspace(gl, ev.shape[0])
    jpet.loglik_grad(gl, ev, rho, s=s, ws=wsl)  # prepares wsl
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(reps):
        jpet.loglik_grad(gl, ev, rho, s=s, ws=wsl, prepared=True)
    torch.cuda.synchronize()
    t_grad = (time.perf_counter() - t0) / reps
    r = rho.clone()
    jpet.mlem_iterate(g, ev, r, 1, s=s, ws=ws, prepared=True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    jpet.mlem_iterate(g, ev, r, reps, s=s, ws=ws, prepared=True)
    torch.cuda.synchronize()
    t_mlem = (time.perf_counter() - t0) / reps
    n = ev.shape[0]
    li = jpet.launch_info(g, n)
    return {"events": n, "pairs_per_pass": n_pairs, "loglik_grad_events_per_s": round(n / t_grad, 1),
            "mlem_events_iterations_per_s": round(n / t_mlem, 1), "ratio": round(t_mlem / t_grad, 3),
            "plans": {"mlem": g.plan, "loglik": gl.plan, "mlem_row_cache": li["row_cache"]}}


def measure_large(jpet, torch):
    """100M events at 1024x1024 px of 0.5 mm (R=450, L=1000, sigma=(5, 30)), 20 iterations, events
    in 8M-event chunks: resident in HBM (prepared once) and, for 2 iterations, streamed from pinned
    host memory (copied and prepared again every iteration)."""
    from jpet_synth import get_workload
    w = get_workload("large1024")
    t0 = time.perf_counter()
    ev_np = w.events(workers=16)
    gen_s = time.perf_counter() - t0
    g = jpet.geometry(**w.geometry())
    s = jpet.sensitivity(g)
    chunk = 8_000_000
    chunks = [torch.from_numpy(ev_np[a:a + chunk]) for a in range(0, len(ev_np), chunk)]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    runner = jpet.ChunkedMLEM(g, chunks, s=s, resident=True)
    torch.cuda.synchronize()
    setup_s = time.perf_counter() - t0
    rho = (s > 0).to(torch.float32)
    runner.iterate(rho, 1)
    torch.cuda.synchronize()
    rho = (s > 0).to(torch.float32)
    t0 = time.perf_counter()
    st = runner.iterate(rho, w.n_iter, want_stats=True)
    torch.cuda.synchronize()
    res_s = time.perf_counter() - t0
    n = len(ev_np)
    pairs = st["n_pairs"]
    del runner
    torch.cuda.empty_cache()
    pinned = [c.pin_memory() for c in chunks]
    stream = jpet.ChunkedMLEM(g, pinned, s=s, resident=False)
    rho = (s > 0).to(torch.float32)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    stream.iterate(rho, 2)
    torch.cuda.synchronize()
    str_s = (time.perf_counter() - t0) / 2
    return {"events": n, "iterations": w.n_iter, "pairs_per_iteration": pairs, "generate_s": round(gen_s, 1),
            "resident_setup_s": round(setup_s, 3),
            "resident_events_iterations_per_s": round(n * w.n_iter / res_s, 1),
            "resident_ms_per_iteration": round(res_s * 1e3 / w.n_iter, 2),
            "streamed_ms_per_iteration": round(str_s * 1e3, 2)}


def measure_workload(jpet, torch, name):
    """A whole reconstruction of a named workload (all its events, its iterations, from rho^0):
    events x iterations / s and ms per iteration.  paper130 is the paper's own setting (R=130,
    L=300, 4 mm pixels, sigma=(10, 40), Appendix A phantom); edge400 is the 400x400 workload with
    sigma_z rising 10% towards the strip ends."""
    from jpet_synth import get_workload
    from paper_1502_07478_amd import tune
    w = get_workload(name)
    ev = torch.from_numpy(w.events()).cuda()
    g = tune.tuned(jpet.geometry(**w.geometry()), ev)  # the plan table's plan, else tuned now
    s = jpet.sensitivity(g)
    rho0 = (s > 0).to(torch.float32)
    ws = jpet.workspace(g, ev.shape[0])
    jpet.prepare(g, ev, ws)
    rho = rho0.clone()
    st = jpet.mlem_iterate(g, ev, rho, 1, s=s, ws=ws, prepared=True, want_stats=True)
    rho.copy_(rho0)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    jpet.mlem_iterate(g, ev, rho, w.n_iter, s=s, ws=ws, prepared=True)
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    n = ev.shape[0]
    return {"events": n, "iterations": w.n_iter, "grid": [w.n_y, w.n_z], "plan": g.plan,
            "pairs_per_iteration": st["n_pairs"],
            "events_iterations_per_s": round(n * w.n_iter / dt, 1), "ms_per_iteration": round(dt * 1e3 / w.n_iter, 3)}


def measure_work_splits(jpet, torch, name="paper130", n_iter=3):
    """The same reconstruction with the event pass split three ways: the planned binned pass, one
    wavefront per event and one thread per event (the paper's GPU "thread" variant): ms per
    iteration each, from rho^0 on a prepared workspace."""
    from jpet_synth import get_workload
    w = get_workload(name)
    ev = torch.from_numpy(w.events()).cuda()
    g = jpet.geometry(**w.geometry())
    s = jpet.sensitivity(g)
    rho0 = (s > 0).to(torch.float32)
    ws = jpet.workspace(g, ev.shape[0])
    jpet.prepare(g, ev, ws)
    out = {"workload": name, "events": ev.shape[0], "iterations": n_iter}
    for split in (None, "wave", "thread"):
        rho = rho0.clone()
        jpet.mlem_iterate(g, ev, rho, 1, s=s, ws=ws, prepared=True, split=split)
        rho.copy_(rho0)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        jpet.mlem_iterate(g, ev, rho, n_iter, s=s, ws=ws, prepared=True, split=split)
        torch.cuda.synchronize()
        out[f"{split or 'binned'}_ms_per_iteration"] = round((time.perf_counter() - t0) * 1e3 / n_iter, 3)
    return out


def measure_event_counts(jpet, torch, name="paper130", counts=(10_000_000, 50_000_000, 100_000_000), n_iter=3):
    """Seconds per iteration of the binned pass against the number of events (10M to 100M) in the
    paper's setting, the layout of its benchmark table: events are prepared once, then n_iter
    iterations from rho^0 are timed."""
    from jpet_synth import get_workload
    w = get_workload(name)
    g = jpet.geometry(**w.geometry())
    s = jpet.sensitivity(g)
    rho0 = (s > 0).to(torch.float32)
    rows = []
    for n in counts:
        ev = torch.from_numpy(w.events(n, workers=16)).cuda()
        ws = jpet.workspace(g, ev.shape[0])
        jpet.prepare(g, ev, ws)
        rho = rho0.clone()
        jpet.mlem_iterate(g, ev, rho, 1, s=s, ws=ws, prepared=True)
        rho.copy_(rho0)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        jpet.mlem_iterate(g, ev, rho, n_iter, s=s, ws=ws, prepared=True)
        torch.cuda.synchronize()
        rows.append({"events": n, "s_per_iteration": round((time.perf_counter() - t0) / n_iter, 5)})
        del ev, ws
        torch.cuda.empty_cache()
    return {"workload": name, "rows": rows}


def _oracle_backprojection(args):
    """Worker of the all-core CPU figure: one event chunk's new-image contribution (no sensitivity
    division), as in the paper's CPU scheme of per-thread images summed at the end."""
    import oracle
    kw, ev, rho = args
    g = oracle.geometry(**kw)
    out, _ = oracle.mlem(g, ev, rho, 1, s=None)
    return out


def cpu_all_cores(w, ev_np, procs=16):
    """The oracle over all host cores: the sample's events split into one chunk per process, the
    chunks' images summed and divided by s (one MLEM iteration), timed around the parallel part."""
    import multiprocessing as mp
    import numpy as np
    import oracle
    procs = max(1, min(procs, os.cpu_count() or 1))
    go = oracle.geometry(**w.geometry())
    so = oracle.sensitivity(go)
    rho0 = oracle.initial_image(so)
    jobs = [(w.geometry(), c, rho0) for c in np.array_split(ev_np, procs)]
    with mp.get_context("spawn").Pool(procs) as pool:
        pool.map(_oracle_backprojection, [(w.geometry(), ev_np[:8], rho0)] * procs)  # start-up
        t0 = time.perf_counter()
        parts = pool.map(_oracle_backprojection, jobs)
        acc = np.sum(parts, axis=0)
        np.divide(acc, so, out=np.zeros_like(acc), where=so > 0)
        dt = time.perf_counter() - t0
    return {"value": round(len(ev_np) / dt, 1), "unit": "events*iterations/s", "cores": procs, "kind": "oracle",
            "sample": f"first {len(ev_np)} events, 1 iteration split over {procs} processes, {dt:.1f} s"}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--workload", default="prod400")
    ap.add_argument("--cpu-events", type=int, default=300_000, help="events in the oracle's timed sample")
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--no-secondary", action="store_true",
                    help="skip the batched (64 instances) and log-likelihood gradient measurements")
    ap.add_argument("--gen-workers", type=int, default=8,
                    help="processes that generate the synthetic events (1: in this process, e.g. under a profiler)")
    ap.add_argument("--calibrate-copy-mib", type=int, default=0,
                    help="before the timed region, one elementwise kernel that reads and writes this many MiB (a "
                         "transfer of known size that scales the memory counters of a profiler run)")
    ap.add_argument("--gradient-only", action="store_true",
                    help="only the log-likelihood gradient against MLEM on grad200 (one JSON line; for profiling "
                         "the log-likelihood pass)")
    ap.add_argument("--extra", action="store_true",
                    help="also measure the batched workload (64 instances), the log-likelihood gradient, the "
                         "paper's setting (work splits, 10M-100M events), the position-dependent sigma_z "
                         "workload and the 1024x1024 workload (100M events in chunks)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py measures one GPU; --gpus {args.gpus} is not supported (this path has no multi-GPU "
              "mode: events would be split across GPUs with one all-reduce of the image per iteration)",
              file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch

    from jpet_synth import get_workload
    from paper_1502_07478_amd import jpet

    if args.gradient_only:
        torch.cuda.set_device(torch.device("cuda:0"))
        print(json.dumps({"gradient": measure_gradient(jpet, torch, args.gen_workers)}), flush=True)
        return

    w = get_workload(args.workload)
    t0 = time.perf_counter()
    ev_np = w.events(workers=args.gen_workers)
    gen_s = time.perf_counter() - t0
    print(f"[bench] {w.name}: {len(ev_np)} events generated in {gen_s:.1f}s", file=sys.stderr, flush=True)

    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    from paper_1502_07478_amd import tune
    g = jpet.geometry(**w.geometry())
    ev = torch.from_numpy(ev_np).to(dev)
    # the event pass's launch plan: the autotuned one (plan table shipped with the package, else
    # timed now on these events), outside the timed region
    t0 = time.perf_counter()
    cached = tune.lookup(g, len(ev_np))
    g = tune.tuned(g, ev)
    tune_s = time.perf_counter() - t0
    plan_info = jpet.launch_info(g, len(ev_np))
    s = jpet.sensitivity(g, device=dev)
    rho0 = (s > 0).to(torch.float32)
    rho = rho0.clone()
    ws = jpet.workspace(g, ev.shape[0], device=dev)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    jpet.prepare(g, ev, ws)
    torch.cuda.synchronize()
    setup_ms = (time.perf_counter() - t0) * 1e3
    st = jpet.mlem_iterate(g, ev, rho, 0, s=s, ws=ws, prepared=True, want_stats=True)
    n_pairs = st["n_pairs"]

    def step():
        rho.copy_(rho0)
        jpet.mlem_iterate(g, ev, rho, w.n_iter, s=s, ws=ws, prepared=True)

    if args.calibrate_copy_mib > 0:
        # an elementwise kernel that reads and writes the given size once each
        nb = args.calibrate_copy_mib << 20
        src_c = torch.ones(nb, dtype=torch.uint8, device=dev)
        dst_c = torch.empty_like(src_c)
        torch.add(src_c, 1, out=dst_c)
        torch.cuda.synchronize()
        del src_c, dst_c
    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    jpet.profile_read()  # discard anything recorded before
    jpet.profile_enable(True)
    # per-step HIP events on the stream the library launches on (the current stream)
    marks = [torch.cuda.Event(enable_timing=True) for _ in range(args.steps + 1)]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    marks[0].record()
    for k in range(args.steps):
        step()
        marks[k + 1].record()
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    step_ms = sorted(marks[k].elapsed_time(marks[k + 1]) for k in range(args.steps))
    median_step_ms = step_ms[len(step_ms) // 2] if len(step_ms) % 2 else 0.5 * (
        step_ms[len(step_ms) // 2 - 1] + step_ms[len(step_ms) // 2])
    launches, pass_ms = jpet.profile_read()
    jpet.profile_enable(False)
    st = jpet.mlem_iterate(g, ev, rho, 0, s=s, ws=ws, prepared=True, want_stats=True)
    assert st["n_unplaced_rows"] == 0

    ms_per_step = elapsed * 1e3 / args.steps
    value = len(ev_np) * w.n_iter * args.steps / elapsed
    avg_pass_s = pass_ms / 1e3 / max(launches, 1)
    achieved = n_pairs / avg_pass_s
    roofline = {
        "bound": "alu",
        "achieved": round(achieved / 1e12, 3),
        "peak": round(PEAK_PAIRS / 1e12, 3),
        "unit": "T pairs/s",
        "frac": round(achieved / PEAK_PAIRS, 4),
        "traffic": MEASURED_TRAFFIC.get(f"{kernel_source_hash()}:{g.plan}"),
        "kernel": "k_event_pass_rings",
        "avg_launch_ms": round(avg_pass_s * 1e3, 4),
        "launches": launches,
        "pairs_per_launch": n_pairs,
        "peak_source": "the pass's arithmetic per pair alone, without LDS, row set-up, masks or idle lanes (microbench)",
        "traffic_source": "rocprofv3 FETCH_SIZE + WRITE_SIZE of these kernel sources and plan, scaled by a device "
                          "copy (profiles/); null when either differs",
        "flops_per_pair": FLOPS_PER_PAIR,
        "achieved_tflops": round(n_pairs * FLOPS_PER_PAIR / avg_pass_s / 1e12, 3),
        "peak_fp32_tflops": PEAK_FP32_TFLOPS,
        "frac_of_fp32_peak": round(n_pairs * FLOPS_PER_PAIR / avg_pass_s / 1e12 / PEAK_FP32_TFLOPS, 4),
    }

    cpu = cpu_all = None
    if not args.no_cpu:
        import oracle
        go = oracle.geometry(**w.geometry())
        so = oracle.sensitivity(go)
        sample = ev_np[: args.cpu_events]
        t0 = time.perf_counter()
        oracle.mlem(go, sample, oracle.initial_image(so), 1, s=so)
        cpu_s = time.perf_counter() - t0
        cpu = {"value": round(len(sample) / cpu_s, 1), "unit": "events*iterations/s", "cores": 1,
               "kind": "oracle", "cpu_model": host_cpu_model(), "host_cpus": os.cpu_count(),
               "sample": f"first {len(sample)} events of the workload, 1 iteration, {cpu_s:.1f} s"}
        cpu_all = cpu_all_cores(w, ev_np[: 4 * args.cpu_events])
        cpu_all["cpu_model"] = host_cpu_model()

    secondary = None

    def measured(key, fn, *a):
        t = time.perf_counter()
        secondary[key] = fn(jpet, torch, *a)
        torch.cuda.empty_cache()
        print(f"[bench] {key}: measured in {time.perf_counter() - t:.1f}s", file=sys.stderr, flush=True)

    if not args.no_secondary or args.extra:
        del ws
        torch.cuda.empty_cache()
        secondary = {}
        measured("batched", measure_batched, args.gen_workers)
        measured("gradient", measure_gradient, args.gen_workers)
    if args.extra:
        measured("paper_setting", measure_workload, "paper130")
        measured("position_dependent_sigma_z", measure_workload, "edge400")
        measured("work_splits", measure_work_splits)
        measured("event_counts", measure_event_counts)
        measured("large", measure_large)

    out = {
        "metric": "events*iterations/s at 400x400 px",
        "value": round(value, 1),
        "unit": "events*iterations/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_per_step, 3),
        "median_ms_per_step": round(median_step_ms, 3),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {
            "workload": (f"{w.name}: R={w.R:g} mm, L={w.L:g} mm, {w.n_y}x{w.n_z} px of {w.pixel:g} mm, "
                         f"sigma_z={w.sigma_z:g} mm, sigma_dl={w.sigma_dl:g} mm, {len(ev_np)} events, "
                         f"{w.n_iter} iterations per step"),
            "events": len(ev_np),
            "iterations_per_step": w.n_iter,
            "pairs_per_iteration": n_pairs,
            "setup_ms": round(setup_ms, 2),
            "plan": {"code": g.plan, "source": "plan table" if cached is not None else f"tuned in {tune_s:.1f} s",
                     "tile_rows": plan_info["tile_rows"], "t_bins": plan_info["t_bins"],
                     "waves": plan_info["waves"], "workgroups_per_cu": plan_info["workgroups_per_cu"],
                     "row_cache": plan_info["row_cache"], "row_segments": plan_info["row_segments"],
                     "accumulator_bits": plan_info["accumulator_bits"],
                     "events_per_workgroup": plan_info["events_per_workgroup"]},
            # the whole job with the one-time preparation of the events counted in
            "end_to_end_events_iterations_per_s": round(len(ev_np) * w.n_iter / ((ms_per_step + setup_ms) / 1e3), 1),
        },
        "roofline": roofline,
        "cpu_baseline": cpu,
    }
    if cpu_all is not None:
        out["cpu_all_cores"] = cpu_all
    if secondary is not None:
        out["secondary"] = secondary
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
