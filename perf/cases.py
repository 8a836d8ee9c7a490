"""The work that users have this library do, case by case, for timing.

Every case is one call, or one short sequence of calls, as a Read Until
program makes them through the package's public entry points:

  one        one read against the whole reference, alone on the device
  batch      a batch of reads: per-read normalisation and scaling, then the
             alignment of every read
  stream     a batch of reads of a serving loop: a resident row is opened for
             each, two chunks of events arrive (the first fixes the read's
             statistics), each extends the rows, the best and the runner-up
             ends are taken for the decision, the rows are given back
  wide       the same for a few reads of a lightly loaded target, whose chunks
             are extended one at a time over the whole device
  events     event detection on complete raw reads
  chunks     event detection on raw samples that arrive chunk by chunk
  reference  preparation of a genome's signal and its device copy

Inputs are simulated on the GPU from the seed alone: uniform random bases, a
6-mer level table of N(90, 12) pA, reads that emit each successive k-mer level
one to three times with N(0, 3.6 pA) noise (half of them; the others are
i.i.d. N(90, 12) pA), raw samples of 4 to 14 per level with N(0, 1.5 pA).
"""
import math

import numpy as np
import torch

import paper_2211_07340_amd as sd

SCALE = 64.0
SMALL, LARGE = 29_903, 5_000_000  # genomes, in bases
WINDOW = 2_000  # runner-up ends lie farther than this from the best (the server's setting)


def listed():
    return [
        # one read, as a latency-bound caller sends it, on a virus-sized and on a bacterial genome
        {"name": "one_small", "kind": "one", "bases": SMALL, "m": 250},
        {"name": "one_large", "kind": "one", "bases": LARGE, "m": 250},
        # a few ragged reads (a flow cell's first minutes): too few to fill the device by reads alone
        {"name": "batch_few", "kind": "batch", "bases": SMALL, "nq": 48, "lo": 20, "hi": 300,
         "dtype": "i16", "tune": False},
        # the benchmark's three batches: equal short reads, very uneven reads, the long reference
        {"name": "batch_equal_f32", "kind": "batch", "bases": SMALL, "nq": 4096, "lo": 250,
         "hi": 250, "dtype": "f32", "tune": True},
        {"name": "batch_uneven", "kind": "batch", "bases": SMALL, "nq": 8192, "lo": 100,
         "hi": 2000, "dtype": "i16", "tune": True},
        {"name": "batch_long_ref", "kind": "batch", "bases": LARGE, "nq": 1024, "lo": 250,
         "hi": 500, "dtype": "i16", "tune": True},
        # the serving loop's batched extension on both genomes
        {"name": "stream_small", "kind": "stream", "bases": SMALL, "ns": 256, "lo": 400,
         "hi": 400, "dtype": "i16"},
        {"name": "stream_large", "kind": "stream", "bases": LARGE, "ns": 256, "lo": 400,
         "hi": 400, "dtype": "i16"},
        # the serving loop at low load
        {"name": "wide_large", "kind": "wide", "bases": LARGE, "ns": 4, "lo": 400, "hi": 400},
        # raw signal: complete reads, and 512 channels' 2,400 samples per 0.1 s
        {"name": "events_reads", "kind": "events", "reads": 4096, "bases": 320, "trim": 50,
         "keep": 250},
        {"name": "events_chunks", "kind": "chunks", "reads": 512, "samples": 2400, "trim": 50,
         "keep": 800},
        # start-up: the reference of a bacterial genome
        {"name": "reference_large", "kind": "reference", "bases": LARGE, "k": 6},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["one", "batch", "batch", "batch", "stream", "stream", "wide", "events",
                       "chunks", "reference"])
    bases = _log(rng, 2_000, LARGE)
    if kind == "one":
        return {"kind": kind, "bases": bases, "m": _log(rng, 20, 2000)}
    if kind == "batch":
        lo = _log(rng, 10, 1000)
        hi = min(4096, _log(rng, lo, 4 * lo))
        most = 4e11 / (2.0 * bases * 0.5 * (lo + hi))  # cells of a pass
        return {"kind": kind, "bases": bases, "nq": _log(rng, 1, max(1.0, min(8192.0, most))),
                "lo": lo, "hi": hi, "dtype": rng.choice(["i16", "f32"]),
                "tune": rng.random() < 0.5}
    if kind == "stream":
        lo = _log(rng, 40, 400)
        hi = _log(rng, lo, 500)
        most = 2e11 / (2.0 * bases * 0.5 * (lo + hi))
        return {"kind": kind, "bases": bases, "ns": _log(rng, 1, max(1.0, min(1024.0, most))),
                "lo": lo, "hi": hi, "dtype": rng.choice(["i16", "i16", "f32"])}
    if kind == "wide":
        lo = _log(rng, 100, 400)
        return {"kind": kind, "bases": bases, "ns": _log(rng, 1, 12), "lo": lo,
                "hi": _log(rng, lo, 500)}
    if kind == "events":
        trim = rng.choice([0, 50, 50, 80])
        return {"kind": kind, "reads": _log(rng, 1, 4096), "bases": _log(rng, 60, 1000),
                "trim": trim, "keep": _log(rng, 50, 1000)}
    if kind == "chunks":
        samples = _log(rng, 300, 4800)
        return {"kind": kind, "reads": _log(rng, 1, 1024), "samples": samples,
                "trim": rng.choice([0, 50]), "keep": max(64, samples // 3)}
    return {"kind": kind, "bases": bases, "k": rng.choice([5, 6, 6, 6, 9])}


# ---- inputs ------------------------------------------------------------------

def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 13)


def _normal(g, shape, mean, sd_):
    return torch.randn(shape, generator=g, device="cuda") * sd_ + mean


def _genome(g, bases, k=6):
    genome = torch.randint(0, 4, (bases,), generator=g, device="cuda", dtype=torch.uint8)
    return genome, _normal(g, (4 ** k,), 90.0, 12.0)


def _currents(genome, table, k=6):
    """Expected current of both strands' k-mers, forward then reverse complement."""
    out = []
    for strand in (genome, 3 - genome.flip(0)):
        n = strand.numel() - k + 1
        idx = torch.zeros(n, dtype=torch.int64, device="cuda")
        for m in range(k):
            idx = idx * 4 + strand[m:m + n]
        out.append(table[idx])
    return torch.cat(out)


def _levels(g, currents, reads, n, repeat):
    """[reads, n] levels: half of the reads walk one strand, emitting each level
    1 .. repeat times; the others are random levels."""
    half = currents.numel() // 2
    steps = torch.rand((reads, n), generator=g, device="cuda") < 2.0 / (repeat + 1)
    pos = torch.cumsum(steps.to(torch.int64), 1)
    room = max(1, half - n)
    start = torch.randint(0, room, (reads, 1), generator=g, device="cuda")
    strand = torch.randint(0, 2, (reads, 1), generator=g, device="cuda")
    on = (start + pos).clamp(max=half - 1) + strand * half
    off = _normal(g, (reads, n), 90.0, 12.0)
    keep = torch.rand((reads, 1), generator=g, device="cuda") < 0.5
    return torch.where(keep, currents[on], off)


def _lengths(which, count, lo, hi):
    """Read lengths, the same for every seed (a plan is made once for a layout)."""
    return np.random.RandomState(which + 7 * lo + hi).randint(lo, hi + 1, count).astype(np.int64)


def _csr(rows, lengths):
    """The first lengths[r] values of each row, concatenated, and their offsets."""
    offs = np.zeros(lengths.size + 1, np.int64)
    np.cumsum(lengths, out=offs[1:])
    keep = torch.arange(rows.shape[1], device="cuda")[None, :] < \
        torch.from_numpy(lengths).cuda()[:, None]
    return rows[keep].contiguous(), offs


def _reads(g, currents, lengths):
    n = int(lengths.max())
    ev = _levels(g, currents, lengths.size, n, 3)
    ev += _normal(g, ev.shape, 0.0, 3.6)
    return _csr(ev, lengths)


def _raw(g, currents, reads, bases):
    """Raw samples of reads of `bases` levels after 30 adaptor levels: values, offsets."""
    lv = torch.cat([_normal(g, (reads, 30), 90.0, 12.0), _levels(g, currents, reads, bases, 1)],
                   1)
    reps = torch.randint(4, 15, lv.shape, generator=g, device="cuda")
    x = torch.repeat_interleave(lv.reshape(-1), reps.reshape(-1))
    x += _normal(g, x.shape, 0.0, 1.5)
    offs = torch.zeros(reads + 1, dtype=torch.int64, device="cuda")
    offs[1:] = torch.cumsum(reps.sum(1), 0)
    return x, offs


def _reference(g, bases, dtype="i16"):
    genome, table = _genome(g, bases)
    z, codes, _ = sd.prepare_reference(genome, table, 6, SCALE)
    values = z if dtype == "f32" else codes
    return sd.Reference(values), values, _currents(genome, table)


def prepare(case, seed):
    g = _generator(seed)
    kind = case["kind"]
    s = {"kind": kind}
    if kind == "one":
        s["ref"], _, cur = _reference(g, case["bases"])
        raw, offs = _reads(g, cur, np.array([case["m"]], np.int64))
        _, s["q"], _ = sd.prepare_queries(raw, torch.from_numpy(offs).cuda(), SCALE)
    elif kind == "batch":
        s["ref"], s["values"], cur = _reference(g, case["bases"], case["dtype"])
        lengths = _lengths(0, case["nq"], case["lo"], case["hi"])
        s["raw"], offs = _reads(g, cur, lengths)
        s["offs"], s["lengths"] = torch.from_numpy(offs).cuda(), lengths
        s["plan"] = sd.Plan(offs, sd.F32 if case["dtype"] == "f32" else sd.I16)
        s["f32"] = case["dtype"] == "f32"
        if case["tune"]:
            z, codes, _ = sd.prepare_queries(s["raw"], s["offs"], SCALE)
            sd.autotune(s["ref"], s["plan"], z if s["f32"] else codes)
    elif kind in ("stream", "wide"):
        dtype = case.get("dtype", "i16")
        s["f32"] = dtype == "f32"
        s["ref"], _, cur = _reference(g, case["bases"], dtype)
        ns = case["ns"]
        first = _lengths(1, ns, case["lo"], case["hi"])
        second = _lengths(2, ns, case["lo"], case["hi"])
        ev = _levels(g, cur, ns, int((first + second).max()), 3)
        ev += _normal(g, ev.shape, 0.0, 3.6)
        a, ao = _csr(ev, first)
        at = torch.from_numpy(first).cuda()[:, None] + \
            torch.arange(int(second.max()), device="cuda")[None, :]
        b, bo = _csr(ev.gather(1, at.clamp(max=ev.shape[1] - 1)), second)
        s["chunks"] = [(a, ao, torch.from_numpy(ao).cuda()), (b, bo, torch.from_numpy(bo).cuda())]
        sd.set_row_budget(48 << 30)
    elif kind == "events":
        genome, table = _genome(g, 100_000)
        s["x"], s["offs"] = _raw(g, _currents(genome, table), case["reads"], case["bases"])
        s["trim"], s["keep"] = case["trim"], case["keep"]
    elif kind == "chunks":
        genome, table = _genome(g, 100_000)
        n, m = case["reads"], case["samples"]
        bases = 2 * m // 4 + 8  # at least 4 samples per level
        s["x"], offs = _raw(g, _currents(genome, table), n, bases)
        s["ranges"] = [torch.stack([offs[:-1], offs[:-1] + c * m], 1).contiguous() for c in (1, 2)]
        s["slots"] = torch.randperm(n, generator=g, device="cuda").to(torch.int32)
        s["states"] = sd.EventStates(n)
        s["trim"], s["keep"] = case["trim"], case["keep"]
    else:
        s["genome"], s["table"] = _genome(g, case["bases"], case["k"])
        s["k"] = case["k"]
    return s


# ---- one pass ----------------------------------------------------------------

def run(s):
    kind = s["kind"]
    if kind == "one":
        cost, end = sd.align_one_wide(s["ref"], s["q"])
        return {"cost": cost, "end": end}
    if kind == "batch":
        z, codes, nsat = sd.prepare_queries(s["raw"], s["offs"], SCALE)
        cost, end = sd.align_batch(s["ref"], s["plan"], z if s["f32"] else codes)
        return {"z": z, "codes": codes, "nsat": nsat, "cost": cost, "end": end}
    if kind in ("stream", "wide"):
        rows = [sd.Stream(s["ref"]) for _ in range(s["chunks"][0][1].size - 1)]
        out, stats = [], None
        for raw, offs, offs_dev in s["chunks"]:
            z, codes, _, stats = sd.prepare_queries_ex(raw, offs_dev, SCALE, stats)
            q = z if s["f32"] else codes
            if kind == "stream":
                out.append(sd.stream_extend(rows, q, offs))
            else:
                out.append([sd.stream_extend_wide(r, q[offs[i]:offs[i + 1]])
                            for i, r in enumerate(rows)])
        best = sd.stream_best_two(rows, WINDOW)
        for r in rows:
            r.close()
        return {"chunks": out, "best": best, "stats": stats}
    if kind == "events":
        events, counts = sd.detect_events(s["x"], s["offs"], s["trim"], s["keep"])
        return {"events": events, "counts": counts}
    if kind == "chunks":
        s["states"].reset(s["slots"])
        return [s["states"].detect(s["x"], r, s["slots"], s["trim"], s["keep"])
                for r in s["ranges"]]
    z, codes, nsat = sd.prepare_reference(s["genome"], s["table"], s["k"], SCALE)
    ref = sd.Reference(codes)
    ref.close()
    return {"z": z, "codes": codes, "nsat": nsat}


def work(case):
    """Bytes: inputs and outputs once, the resident rows once for each chunk
    that reads or writes them.  Operations: five per cell (subtract, absolute
    value, two comparisons, add); events: the two t statistics of a sample."""
    kind = case["kind"]
    n = 2 * (case.get("bases", 0) - 5)
    if kind == "one":
        return {"bytes": 2 * n + 2 * case["m"] + 8, "flops": 5.0 * n * case["m"]}
    if kind == "batch":
        values = 0.5 * (case["lo"] + case["hi"]) * case["nq"]
        size = 4 if case["dtype"] == "f32" else 2
        return {"bytes": size * n + values * (4 + 4 + 2) + 16 * case["nq"],
                "flops": 5.0 * n * values}
    if kind in ("stream", "wide"):
        values = (case["lo"] + case["hi"]) * case["ns"]  # both chunks
        # rows: written by each chunk, read by the second and by the search
        return {"bytes": 4.0 * n * 4 * case["ns"] + 10 * values, "flops": 5.0 * n * values}
    if kind == "events":
        samples = min(case["bases"] + 30, 1.2 * (case["trim"] + case["keep"])) * 9 * case["reads"]
        return {"bytes": 4 * samples + 4 * case["reads"] * case["keep"], "flops": 70.0 * samples}
    if kind == "chunks":
        samples = 2 * case["samples"] * case["reads"]
        return {"bytes": 4 * samples + 8 * case["reads"] * case["keep"], "flops": 70.0 * samples}
    n = 2 * (case["bases"] - case["k"] + 1)
    return {"bytes": case["bases"] + n * (4 + 2 + 2 + 4), "flops": 6.0 * n}


# ---- the same in 64 bits -----------------------------------------------------

def _zscores(raw, offs):
    """Each read's z-scores in float64."""
    x = raw.double().cpu().numpy()
    o = offs.cpu().numpy()
    z = np.empty_like(x)
    for a, b in zip(o[:-1], o[1:]):
        v = x[a:b]
        d = v.std()
        z[a:b] = (v - v.mean()) / d if d > 0 else 0.0
    return z


def _costs(z, lengths, ref):
    """Subsequence-DTW costs in float64, an anti-diagonal of every read at a time."""
    nq, m, n = lengths.size, int(lengths.max()), ref.numel()
    offs = np.concatenate([[0], np.cumsum(lengths)])
    x = torch.zeros((nq, m), dtype=torch.float64, device="cuda")
    for r in range(nq):
        x[r, :lengths[r]] = torch.from_numpy(z[offs[r]:offs[r + 1]]).cuda()
    inf = torch.tensor(math.inf, dtype=torch.float64, device="cuda")
    # row i of diagonal t is the cell (i, t - i); row 0 is the free start
    y = torch.cat([inf.expand(m), ref.double(), inf.expand(m)]).flip(0)
    d1 = torch.full((nq, m + 1), math.inf, dtype=torch.float64, device="cuda")
    d2 = d1.clone()
    d1[:, 0] = d2[:, 0] = 0.0
    last = torch.from_numpy(lengths).cuda()[:, None]
    best = torch.full((nq, 1), math.inf, dtype=torch.float64, device="cuda")
    for t in range(n + m - 1):
        cols = y[n + m - 1 - t:n + 2 * m - 1 - t]  # column t - i of each row i
        new = torch.minimum(torch.minimum(d1[:, :-1], d2[:, :-1]), d1[:, 1:])
        new = torch.nan_to_num((x - cols).abs() + new, nan=math.inf, posinf=math.inf)
        d2, d1 = d1, torch.nn.functional.pad(new, (1, 0))
        best = torch.minimum(best, d1.gather(1, last))
    return best[:, 0]


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        s = prepare(dict(case, tune=False), seed)
        z = _zscores(s["raw"], s["offs"])
        n, m = s["values"].numel(), int(s["lengths"].max())
        steps, cells = n + m, float(s["lengths"].size) * m
        cost = None
        if s["f32"] and steps * (6e-5 + cells * 6e-11) < 12 and s["lengths"].size <= 4096:
            cost = _costs(z, s["lengths"], s["values"])
        return {"z": z, "codes": None, "nsat": None, "cost": cost, "end": None}
    if kind in ("stream", "wide"):
        s = prepare(case, seed)
        raw, offs, _ = s["chunks"][0]
        x = raw.double().cpu().numpy()
        stats = [[x[a:b].mean(), x[a:b].std()] for a, b in zip(offs[:-1], offs[1:])]
        return {"chunks": None, "best": None, "stats": np.array(stats)}
    if kind == "reference":
        s = prepare(case, seed)
        x = _currents(s["genome"], s["table"], s["k"]).double()
        return {"z": (x - x.mean()) / x.std(unbiased=False), "codes": None, "nsat": None}
    return None
