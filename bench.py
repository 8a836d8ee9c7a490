"""sDTW benchmark on one MI355X: prints one JSON line.

A step is one pass of the hot path over one batch: per-read normalisation and
fixed-point scaling of the raw events (sdtw_prepare_queries) followed by the
batched alignment of every read against the reference (sdtw_align_batch).
The reference is prepared once on the device (sdtw_prepare_reference) before
the timed region; all inputs are resident in HBM when timing starts.

Workload (default, the largest batch): 1,024 reads of 250-500 events against
the 9,999,990-value forward+reverse signal of a 5,000,000-base genome
(seeded synthetic data; the reference is streamed through the kernel in
column tiles), int16 inputs with 32-bit accumulation.  The 4,096-read and
8,192-read workloads against the 29,903-base genome are measured in the same
run (`extras.workloads`), in both number formats.

`value` is GCUPS (cells = sum over reads of M x N, per second of step time).
`extras.end_to_end` gives the same pass with its host transfers (inputs up
from pinned host memory, results back), which `value` leaves out.
The roofline object reports the alignment kernel's cell rate, timed with HIP
events on the launch stream, against the VALU roof of the chip: 256 CUs x 4
SIMDs x 2.4 GHz, where a SIMD spends 4 cycles on a full-rate 32-bit VALU
instruction of a 64-lane wave (min, max, min3, sad; 16 lanes per cycle) and 2
cycles on a float32 add/sub (the published 157.3 TFLOP/s float32 vector peak
is twice the full rate; the issue-rate measurements are in
profiles/valu_issue_rates_gfx950.md).  A cell costs v_min3_u32 + v_sad_u32 =
8 SIMD cycles per 64 cells on the int16 path and v_sub_f32 + v_min3_u32 +
v_add_f32 = 2 + 4 + 2 = 8 on the float32 path: 19.66 TCUPS for both.
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
# The serving leg runs several HIP streams per target; HIP maps streams onto
# this many hardware queues round-robin (4 by default), and two streams on one
# queue run in order, so a short-reference batch could wait behind a
# long-reference one.  Eight queues give every stream its own.  Read at HIP
# initialisation, so set before torch touches the device (and over any
# smaller value the environment holds).
if int(os.environ.get("GPU_MAX_HW_QUEUES", "4")) < 8:
    os.environ["GPU_MAX_HW_QUEUES"] = "8"

CUS, SIMDS_PER_CU, CLOCK_GHZ = 256, 4, 2.4
# SIMD cycles per 64 cells (one wave-wide row of a strip column): int16
# v_min3_u32 + v_sad_u32, float32 v_sub_f32 + v_min3_u32 + v_add_f32 |.|.
# Full-rate 32-bit instructions take 4 cycles per 64-lane wave, float32
# add/subtract 2 (the measured rates: profiles/valu_issue_and_lds_rates_gfx950.md,
# `python bench_experiments.py issue`).
SIMD_CYCLES_PER_64_CELLS = {"i16": 4 + 4, "f32": 2 + 4 + 2}


# HBM bytes per alignment call (halo and sweep), from the rocprofv3 FETCH_SIZE
# and WRITE_SIZE passes summarised in
# profiles/counters_k_rows_i16_1024xU250-500_vs_9999990.md (mean of the timed
# calls), scaled by what the counter reads for a plain device copy of known
# size (factors 1.9998 and 1.0000), keyed by workload, valid only without a
# launch shape of the caller's and while the sources that make and cut the
# launch are the ones measured; otherwise `traffic` is null.
TRAFFIC_SOURCES = ("rows.h", "cells.h", "cut.h", "api.hip")
MEASURED_TRAFFIC = {
    ("1024 reads M~U[250,500] vs 5,000,000-base genome", "i16"): {
        "fetch_bytes": 5935129372, "write_bytes": 184405120,
        "sha256": "987caecf6abc5b358482997e02e3641bf4d38fba8ca4507deee11cda530b7467"},
}


_T0 = time.perf_counter()


def progress(msg: str):
    """One line on stderr per stage (the JSON line alone goes to stdout)."""
    print(f"bench [{time.perf_counter() - _T0:7.1f} s] {msg}", file=sys.stderr, flush=True)


def measured_traffic(workload: str, dtype: str, shaped: bool):
    import hashlib
    m = MEASURED_TRAFFIC.get((workload, dtype))
    if m is None or shaped:
        return None
    h = hashlib.sha256()
    for name in TRAFFIC_SOURCES:
        with open(os.path.join(ROOT, "paper_2211_07340_amd", "csrc", name), "rb") as f:
            h.update(f.read())
    if h.hexdigest() != m["sha256"]:
        return None
    return m["fetch_bytes"] + m["write_bytes"]


def launch_shape(plan, reads, shaped: bool = False):
    """The shape a plan's reads are launched in: its own only where one was set or
    reads are longer than the row-lane kernel takes (the library cuts its launch)."""
    if shaped or int(reads.lengths.max()) > 2048:
        return plan.config
    return {"launch": "row-lane kernel, cut by the library's model"}


def valu_peak_tcups(dtype: str) -> float:
    return CUS * SIMDS_PER_CU * CLOCK_GHZ * 1e9 * 64 / SIMD_CYCLES_PER_64_CELLS[dtype] / 1e12


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--config", type=int, default=3, choices=[1, 2, 3])
    ap.add_argument("--dtype", default="i16", choices=["i16", "f32"])
    ap.add_argument("--strip", type=int, default=0)
    ap.add_argument("--chains", type=int, default=0)
    ap.add_argument("--waves", type=int, default=0)
    ap.add_argument("--bands", type=int, default=0, help="waves per read (row bands): 1, 2, 4")
    ap.add_argument("--band-rows", type=int, default=-1,
                    help="target rows per band (0: as many bands as fit)")
    ap.add_argument("--no-autotune", action="store_true",
                    help="keep the plan's default launch shape instead of autotuning it")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-extras", action="store_true",
                    help="skip the float32 and one-read-per-launch comparison legs")
    ap.add_argument("--cpu-sample", type=int, default=0,
                    help="reads in the oracle's timed sample (0: sized for ~10 s)")
    ap.add_argument("--serve-seconds", type=float, default=20.0,
                    help="measured seconds of the streaming server leg (0: skip)")
    ap.add_argument("--serve-warmup", type=float, default=5.0)
    ap.add_argument("--serve-channels", type=int, default=512)
    ap.add_argument("--serve-recompute-seconds", type=float, default=10.0)
    ap.add_argument("--serve-low-channels", type=int, default=64,
                    help="serving: a second, low-load incremental run at this many channels, "
                         "8 s after 3 s (0: none)")
    ap.add_argument("--serve-small-only", action="store_true",
                    help="serve the 29,903-base target only")
    return ap.parse_args()


def main():
    args = parse()
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (got --gpus {args.gpus}); the sDTW path "
              "is built and measured for a single MI355X", file=sys.stderr)
        sys.exit(2)
    import torch

    import synth
    import paper_2211_07340_amd as sd

    dev = torch.device("cuda:0")
    w = synth.workload(args.config)
    reads = w.reads
    nq = reads.nq
    dt = sd.I16 if args.dtype == "i16" else sd.F32

    progress(f"{w.name}: preparing the reference")
    # one-time reference preparation on the device (section 4.1)
    g = torch.from_numpy(w.genome).to(dev)
    tab = torch.from_numpy(w.table).to(dev)
    zref, cref, _ = sd.prepare_reference(g, tab, w.k, 64.0)
    ref = sd.Reference(cref if dt == sd.I16 else zref)
    N = ref.n
    raw = torch.from_numpy(reads.values).to(dev)
    offs_dev = torch.from_numpy(reads.offsets).to(dev)
    plan = sd.Plan(reads.offsets, dt)
    tune_ms = None
    shaped = bool(args.strip or args.chains or args.waves or args.bands or args.band_rows >= 0)
    if shaped:
        plan.set_config(args.strip, args.chains, args.waves, args.bands, args.band_rows)
    elif not args.no_autotune:
        # launch shape picked by the library's autotuner on this batch (on the
        # first 2^17 reference columns), outside the timed region
        z0, c0, _ = sd.prepare_queries(raw, offs_dev, 64.0)
        torch.cuda.synchronize()
        t_tune = time.perf_counter()
        sd.autotune(ref, plan, c0 if dt == sd.I16 else z0)
        tune_ms = round((time.perf_counter() - t_tune) * 1e3, 1)
    cost = torch.empty(nq, dtype=torch.int32 if dt == sd.I16 else torch.float32, device=dev)
    end = torch.empty(nq, dtype=torch.int32, device=dev)
    cells = float(reads.lengths.sum()) * N

    stream = torch.cuda.current_stream()

    def step(ev=None):
        z, codes, _ = sd.prepare_queries(raw, offs_dev, 64.0)
        q = codes if dt == sd.I16 else z
        if ev is not None:
            ev[0].record(stream)
        sd.align_batch(ref, plan, q, cost, end)
        if ev is not None:
            ev[1].record(stream)

    progress(f"{launch_shape(plan, reads, shaped)}; {args.warmup} warm-up and {args.steps} timed steps")
    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    evs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
           for _ in range(args.steps)]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for k in range(args.steps):
        step(evs[k])
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    ms_step = (t1 - t0) * 1e3 / args.steps
    kern_ms = float(np.median([a.elapsed_time(b) for a, b in evs]))
    gcups = cells / (ms_step * 1e-3) / 1e9
    kern_tcups = cells / (kern_ms * 1e-3) / 1e12
    peak = valu_peak_tcups(args.dtype)
    pcfg = launch_shape(plan, reads, shaped)

    out = {
        "metric": "sDTW GCUPS at 1 GPU (% VALU peak)",
        "value": round(gcups, 1),
        "unit": "GCUPS",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(ms_step, 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "i16/i32" if dt == sd.I16 else "f32",
        "data": "synthetic (seeded genome, stand-in 6-mer pore model, simulated reads)",
        "config": {"workload": w.name, "reads": nq, "query_values": int(reads.values.size),
                   "reference_values": N, "cells_per_step": cells,
                   **pcfg, "autotune_ms": tune_ms},
        "reads_per_s": round(nq / (ms_step * 1e-3), 1),
        "pct_valu_peak": round(100 * gcups / (peak * 1e3), 2),
        "roofline": {"bound": "alu", "kernel": "sdtw_align_batch",
                     "achieved": round(kern_tcups, 3), "peak": round(peak, 3),
                     "unit": "TCUPS", "frac": round(kern_tcups / peak, 4),
                     "kernel_ms": round(kern_ms, 4),
                     "traffic": measured_traffic(w.name, args.dtype, shaped)},
    }

    progress(f"{kern_ms:.2f} ms per alignment launch ({kern_tcups / peak:.3f} of the roof)")
    if not args.no_extras:
        out["extras"] = extras(sd, torch, dev, w, reads, zref, cref, args, stream)
        # about two seconds of replays each
        reps = max(3, min(args.steps, int(2000 / max(ms_step, 1e-3))))
        out["extras"]["hip_graph"] = graph_step(sd, torch, step, cost, end, reps)
        out["extras"]["end_to_end"] = end_to_end(sd, torch, dev, reads, ref, plan, dt, cells,
                                                 reps)

    if args.serve_seconds > 0:
        progress("serving")
        out["serving"] = serving(torch, dev, args.serve_seconds, args.serve_warmup,
                                 args.serve_channels, args.serve_recompute_seconds,
                                 large=not args.serve_small_only,
                                 low_channels=args.serve_low_channels)

    if not args.no_cpu_baseline:
        progress("CPU baseline (the oracle)")
        out["cpu_baseline"] = cpu_baseline(w, reads, args)
    progress("done")
    print(json.dumps(out), flush=True)


def graph_step(sd, torch, step, cost, end, steps):
    """The same step captured once in a HIP graph and replayed: time per
    replay, and whether every replay's outputs equal the eager step's."""
    step()
    torch.cuda.synchronize()
    want = (cost.clone(), end.clone())
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step()
    g.replay()
    torch.cuda.synchronize()
    same = bool(torch.equal(cost, want[0]) and torch.equal(end, want[1]))
    t0 = time.perf_counter()
    for _ in range(steps):
        g.replay()
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) * 1e3 / steps
    same = same and bool(torch.equal(cost, want[0]) and torch.equal(end, want[1]))
    return {"ms_per_step": round(ms, 4), "replays": steps + 1, "equal_to_eager": same}


def end_to_end(sd, torch, dev, reads, ref, plan, dt, cells, reps):
    """The step with its host transfers: the raw events and offsets go up from
    pinned host memory, the step runs, cost and end come back to pinned host
    memory; host wall time per pass until the results are on the host
    (median).  Not the headline value, whose inputs are resident."""
    h_raw = torch.empty(reads.values.size, dtype=torch.float32, pin_memory=True)
    h_raw.copy_(torch.from_numpy(reads.values))
    h_offs = torch.empty(reads.offsets.size, dtype=torch.int64, pin_memory=True)
    h_offs.copy_(torch.from_numpy(reads.offsets))
    cdt = torch.int32 if dt == sd.I16 else torch.float32
    h_cost = torch.empty(reads.nq, dtype=cdt, pin_memory=True)
    h_end = torch.empty(reads.nq, dtype=torch.int32, pin_memory=True)
    d_raw = torch.empty(h_raw.shape, dtype=torch.float32, device=dev)
    d_offs = torch.empty(h_offs.shape, dtype=torch.int64, device=dev)
    d_cost = torch.empty(reads.nq, dtype=cdt, device=dev)
    d_end = torch.empty(reads.nq, dtype=torch.int32, device=dev)
    cur = torch.cuda.current_stream()

    def run():
        d_raw.copy_(h_raw, non_blocking=True)
        d_offs.copy_(h_offs, non_blocking=True)
        z, codes, _ = sd.prepare_queries(d_raw, d_offs, 64.0)
        sd.align_batch(ref, plan, codes if dt == sd.I16 else z, d_cost, d_end)
        h_cost.copy_(d_cost, non_blocking=True)
        h_end.copy_(d_end, non_blocking=True)
        cur.synchronize()

    run()
    times = []
    for _ in range(reps):
        t0 = time.perf_counter()
        run()
        times.append(time.perf_counter() - t0)
    ms = float(np.median(times)) * 1e3
    up = reads.values.size * 4 + reads.offsets.size * 8
    return {"ms": round(ms, 4), "gcups": round(cells / (ms * 1e-3) / 1e9, 1),
            "h2d_bytes": int(up), "d2h_bytes": int(reads.nq * 8), "passes": reps}


def workload_leg(sd, torch, dev, c, stream, reps=10):
    """Workload c in both number formats: device preparation, autotuned launch
    shape, median kernel time of `reps` launches (HIP events on the launch
    stream)."""
    import synth
    w = synth.workload(c)
    reads = w.reads
    g = torch.from_numpy(w.genome).to(dev)
    tab = torch.from_numpy(w.table).to(dev)
    zref, cref, _ = sd.prepare_reference(g, tab, w.k, 64.0)
    raw = torch.from_numpy(reads.values).to(dev)
    offs_dev = torch.from_numpy(reads.offsets).to(dev)
    z, codes, _ = sd.prepare_queries(raw, offs_dev, 64.0)
    out = {"workload": w.name, "reads": int(reads.nq), "reference_values": int(zref.numel())}
    for name, dt, rv, q in (("i16", sd.I16, cref, codes), ("f32", sd.F32, zref, z)):
        ref = sd.Reference(rv)
        plan = sd.Plan(reads.offsets, dt)
        sd.autotune(ref, plan, q)
        cost, end = sd.align_batch(ref, plan, q)
        ms = _median_event_ms(torch, stream, lambda: sd.align_batch(ref, plan, q, cost, end),
                              reps)
        cells = float(reads.lengths.sum()) * ref.n
        out[name] = {"kernel_ms": round(ms, 4), "gcups": round(cells / ms / 1e6, 1),
                     "frac_valu_peak": round(cells / ms / 1e9 / valu_peak_tcups(name), 4),
                     **launch_shape(plan, reads)}
        plan.close()
        ref.close()
    return out


def scale_sweep(sd, torch, dev):
    """Accuracy against the fixed-point scale (section 6): for scales 2 ..
    256, the share of the 4,096 reads of workload 1 whose int16-path end
    equals the float32-path end, and the saturated values."""
    import synth
    w = synth.workload(1)
    reads = w.reads
    g = torch.from_numpy(w.genome).to(dev)
    tab = torch.from_numpy(w.table).to(dev)
    raw = torch.from_numpy(reads.values).to(dev)
    offs = torch.from_numpy(reads.offsets).to(dev)
    zref, _, _ = sd.prepare_reference(g, tab, w.k, 64.0)
    fref = sd.Reference(zref)
    zq, _, _ = sd.prepare_queries(raw, offs, 64.0)
    fplan = sd.Plan(reads.offsets, sd.F32)
    _, fend = sd.align_batch(fref, fplan, zq)
    torch.cuda.synchronize()
    fend = fend.cpu().numpy()
    on = reads.on_target
    rows = []
    for s in (2, 4, 8, 16, 32, 64, 128, 256):
        _, cref, rsat = sd.prepare_reference(g, tab, w.k, float(s))
        _, cq, qsat = sd.prepare_queries(raw, offs, float(s))
        iref = sd.Reference(cref)
        iplan = sd.Plan(reads.offsets, sd.I16)
        _, iend = sd.align_batch(iref, iplan, cq)
        torch.cuda.synchronize()
        iend = iend.cpu().numpy()
        same = iend == fend
        rows.append({"scale": s,
                     "pct_end_equal_all": round(100 * float(same.mean()), 2),
                     "pct_end_equal_on_target": round(100 * float(same[on].mean()), 2),
                     "pct_end_within_10_on_target": round(
                         100 * float((np.abs(iend - fend) <= 10)[on].mean()), 2),
                     "saturated_reference_values": int(rsat),
                     "saturated_query_values": int(qsat)})
        iplan.close()
        iref.close()
    fplan.close()
    fref.close()
    return {"workload": w.name, "reads": int(reads.nq), "by_scale": rows}


def extras(sd, torch, dev, w, reads, zref, cref, args, stream):
    """The other number format, the other workloads, the one-read-per-launch
    baseline, the whole-device single query, event detection and the
    accuracy-against-scale sweep."""
    res = {}
    other = "f32" if args.dtype == "i16" else "i16"
    progress(f"extras: {other}")
    dt = sd.F32 if other == "f32" else sd.I16
    ref = sd.Reference(zref if dt == sd.F32 else cref)
    raw = torch.from_numpy(reads.values).to(dev)
    offs_dev = torch.from_numpy(reads.offsets).to(dev)
    z, codes, _ = sd.prepare_queries(raw, offs_dev, 64.0)
    q = z if dt == sd.F32 else codes
    plan = sd.Plan(reads.offsets, dt)
    sd.autotune(ref, plan, q)
    cost, end = sd.align_batch(ref, plan, q)
    reps = 5 if ref.n > 1_000_000 else 20
    ms = _median_event_ms(torch, stream, lambda: sd.align_batch(ref, plan, q, cost, end), reps)
    cells = float(reads.lengths.sum()) * ref.n
    res[other] = {"kernel_ms": round(ms, 4), "gcups": round(cells / ms / 1e6, 1),
                  "frac_valu_peak": round(cells / ms / 1e9 / valu_peak_tcups(other), 4),
                  **launch_shape(plan, reads)}
    plan.close()
    # the other batch workloads, both number formats
    res["workloads"] = []
    for c in (1, 2, 3):
        if c != args.config:
            progress(f"extras: workload {c}")
            res["workloads"].append(workload_leg(sd, torch, dev, c, stream))
    progress("extras: one read per launch, whole device, event detection, scales")
    # one read per launch with the single-wave kernel, on the main dtype
    dt0 = sd.I16 if args.dtype == "i16" else sd.F32
    ref0 = sd.Reference(cref if dt0 == sd.I16 else zref)
    q0 = codes if dt0 == sd.I16 else z
    n1 = min(256 if ref0.n < 1_000_000 else 2, reads.nq)
    offs = reads.offsets
    sd.align_one(ref0, q0[offs[0]:offs[1]])
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for r in range(n1):
        sd.align_one(ref0, q0[offs[r]:offs[r + 1]])
    torch.cuda.synchronize()
    t = time.perf_counter() - t0
    c1 = float(reads.lengths[:n1].sum()) * ref0.n
    res["plain_one_read_per_launch"] = {"reads": n1, "ms_per_read": round(t * 1e3 / n1, 4),
                                        "gcups": round(c1 / t / 1e9, 2)}
    if dt0 == sd.I16:
        # the first read over every compute unit (row scans with look-back)
        q1 = q0[offs[0]:offs[1]]
        m1 = int(offs[1] - offs[0])
        ms1 = _median_event_ms(torch, stream, lambda: sd.align_one_wide(ref0, q1), 20)
        res["single_query_whole_device"] = {
            "query_values": m1, "reference_values": ref0.n, "ms": round(ms1, 4),
            "paper_accelerator_model_ms": round((ref0.n + m1 - 1) / 1e8 * 1e3, 4)}
        if ref0.n > 1_000_000:
            res["stream_extension"] = stream_extension_leg(sd, torch, dev, ref0, stream)
    # pre-processing on the device: event detection and trimming of raw reads
    import synth
    sg = synth.make_genome(synth.SMALL_GENOME, synth.SMALL_GENOME)
    rr = synth.simulate_raw(sg, w.table, 4096, 320, 0.5, 4242)
    xr = torch.from_numpy(rr.values).to(dev)
    xo = torch.from_numpy(rr.offsets).to(dev)
    ms_ev = _median_event_ms(torch, stream, lambda: sd.detect_events(xr, xo, 50, 250), 5)
    res["event_detection"] = {"raw_reads": rr.nreads, "raw_samples": int(rr.values.size),
                              "trim": 50, "keep": 250, "ms": round(ms_ev, 4),
                              "reads_per_s": round(rr.nreads / (ms_ev * 1e-3), 1)}
    res["accuracy_vs_scale"] = scale_sweep(sd, torch, dev)
    ref0.close()
    ref.close()
    return res


def stream_extension_leg(sd, torch, dev, ref, stream, k=256, m=400):
    """Resident-row extension on the long reference: k streams (one per CU
    on an MI355X) extended by an m-value chunk each in one batched launch
    (HIP events on the launch stream, median of three after the first
    chunk), and two such batches issued at once on two HIP streams
    (host clock), as the Read Until server keeps two per target in flight."""
    progress("extras: resident-row extension")
    budget0 = sd.row_budget_info()[0]
    sd.set_row_budget(max(budget0, 2 * k * 4 * (ref.n + 8192) + (1 << 30)))
    rng = np.random.default_rng(5)
    streams = [sd.Stream(ref) for _ in range(2 * k)]
    offs = np.arange(k + 1, dtype=np.int64) * m
    qa = torch.from_numpy(rng.integers(-300, 300, size=k * m).astype(np.int16)).to(dev)
    qb = torch.from_numpy(rng.integers(-300, 300, size=k * m).astype(np.int16)).to(dev)
    sd.stream_extend(streams[k:], qb, offs)  # first chunk of the second set
    torch.cuda.synchronize()
    ms = _median_event_ms(torch, stream, lambda: sd.stream_extend(streams[:k], qa, offs,
                                                                  stream=stream), 3)
    # the server's own HIP streams: a stream created beyond the hardware
    # queues shares one with an older stream, and the serving leg that
    # follows would then find its streams serialised
    from paper_2211_07340_amd import server as srv
    hs = srv._server_streams(torch, 0, 2)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    sd.stream_extend(streams[:k], qa, offs, stream=hs[0])
    sd.stream_extend(streams[k:], qb, offs, stream=hs[1])
    torch.cuda.synchronize()
    two = (time.perf_counter() - t0) * 1e3
    for st in streams:
        st.close()
    torch.cuda.synchronize()
    sd.row_pool_trim()  # about 20 GB of rows back to the device
    sd.set_row_budget(budget0)
    cells = float(k) * m * ref.n
    peak = valu_peak_tcups("i16")
    return {"chunks": k, "chunk_values": m, "reference_values": ref.n,
            "one_batch_ms": round(ms, 3), "frac_valu_peak": round(cells / ms / 1e9 / peak, 4),
            "two_batches_at_once_ms": round(two, 3),
            "two_batches_frac_valu_peak": round(2 * cells / two / 1e9 / peak, 4)}


def _median_event_ms(torch, stream, fn, reps):
    """Median device time of fn() (HIP events on the launch stream) after one
    untimed call."""
    fn()
    torch.cuda.synchronize()
    out = []
    for _ in range(reps):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record(stream)
        fn()
        b.record(stream)
        b.synchronize()
        out.append(a.elapsed_time(b))
    return float(np.median(out))


def serving_targets(torch, dev, pool: int = 512, seed: int = 4400, large: bool = True):
    """Workload 4's two targets: the 29,903-base and the 5,000,000-base genome,
    each with a pool of 2,000-event reads (50% on-target)."""
    import synth
    from paper_2211_07340_amd import server as srv
    table = synth.make_level_table()
    specs = []
    genomes = [("29,903-base", synth.SMALL_GENOME)]
    if large:
        genomes.append(("5,000,000-base", synth.LARGE_GENOME))
    for i, (name, L) in enumerate(genomes):
        genome = synth.make_genome(L, L)
        rd = synth.simulate_reads(genome, table, np.full(pool, 2000), 0.5, seed + i)
        raws = [rd.values[rd.offsets[r]:rd.offsets[r + 1]] for r in range(pool)]
        specs.append((name, genome, table, raws, rd.on_target))
    return srv.make_targets(specs, dev)


def serving(torch, dev, seconds: float, warmup: float, channels: int, recompute_s: float,
            large: bool = True, low_channels: int = 0):
    """Streaming Read Until: incremental extension, then recompute from
    scratch; then incremental extension at a low load, where small batches
    of long-reference chunks go over the whole device one chunk at a time."""
    from paper_2211_07340_amd import server as srv
    targets = serving_targets(torch, dev, large=large)
    cfg = srv.ServerConfig(channels=channels, row_budget_bytes=64 << 30)
    inc = srv.ReadUntilServer(targets, cfg, mode="extend")
    inc.calibrate()
    out = {"workload": f"{channels} channels, 400-event chunks every 0.1 s, reads to "
                       f"{cfg.max_events} events, targets " +
                       " and ".join(t.name for t in targets) + " (50/50)",
           "incremental": inc.run(seconds, warmup)}
    if recompute_s > 0:
        rec = srv.ReadUntilServer(targets, cfg, mode="recompute")
        out["recompute"] = rec.run(recompute_s, min(warmup, 2.0))
    if low_channels > 0:
        low = srv.ReadUntilServer(
            targets, srv.ServerConfig(channels=low_channels, row_budget_bytes=64 << 30),
            mode="extend")
        cal = low.calibrate()
        out["low_load"] = {"channels": low_channels,
                           "wide_max": {k: v["wide_max"] for k, v in cal.items()},
                           "incremental": low.run(8.0, 3.0)}
    for t in targets:
        t.ref.close()
    return out


def cpu_baseline(w, reads, args):
    """The oracle, untouched, on the host cores over a bounded sample."""
    import oracle
    z, codes, _ = oracle.prepare_reference(w.genome, w.table, w.k)
    qz, qc, _ = oracle.prepare_queries(reads.values, reads.offsets)
    # a one-GPU host here gives each GPU 16 cores, whatever the affinity
    # mask shows
    cores = min(16, len(os.sched_getaffinity(0)))
    kind = oracle.I64 if args.dtype == "i16" else oracle.F32
    q = qc if args.dtype == "i16" else qz
    r = codes if args.dtype == "i16" else z
    if args.cpu_sample:
        n = args.cpu_sample
    else:  # 1e10 cells per core: about 10-15 s at the oracle's ~0.7 GCUPS per core
        per_read = reads.lengths.astype(np.float64) * r.size
        n = int(np.searchsorted(np.cumsum(per_read), 1e10 * cores)) + 1
        n = max(1, min(reads.nq, n))
    idx = np.arange(n)
    threads = min(cores, n)
    t0 = time.perf_counter()
    _, _, used = oracle.batch(kind, q, reads.offsets, r, index=idx, nthreads=threads)
    t = time.perf_counter() - t0
    cells = float(reads.lengths[:n].sum()) * r.size
    return {"value": round(cells / t / 1e9, 3), "unit": "GCUPS", "cores": used,
            "kind": "oracle", "seconds": round(t, 2),
            "sample": f"first {n} of the {reads.nq} reads of the same batch "
                      f"({cells:.3g} cells), {'int64' if kind == oracle.I64 else 'float32'} "
                      f"oracle, one read per task on {used} threads"}


if __name__ == "__main__":
    main()
