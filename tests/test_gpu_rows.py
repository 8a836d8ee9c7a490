"""The row-lane kernel (batches, chunks and single reads without a launch
shape of their own) against the oracle, where it can go wrong: rows per lane
and lanes per read at their edges, several reads in a wave, references shorter
than a block of steps and ragged against the four columns of a step, column
segments whose left column settles at once, late or never.  Bit-exact in both
formats.
"""
import sys

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
sd = pytest.importorskip("paper_2211_07340_amd")


def note(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sd.load_library()
    return torch.device("cuda:0")


def values(rng, n, dt, spread=3000):
    v = rng.integers(-spread, spread, size=n)
    return v.astype(np.int16) if dt == "i16" else (v / 64).astype(np.float32)


def check_batch(dev, ref_np, reads, dt):
    q, offs = synth.csr(reads)
    q = q.astype(ref_np.dtype)
    kind, code = (oracle.I64, sd.I16) if dt == "i16" else (oracle.F32, sd.F32)
    want_c, want_e, _ = oracle.batch(kind, q, offs, ref_np)
    ref = sd.Reference(torch.from_numpy(ref_np).to(dev))
    plan = sd.Plan(offs, code)
    for _ in range(2):  # the second call finds the scratch as the first left it
        cost, end = sd.align_batch(ref, plan, torch.from_numpy(q).to(dev))
        torch.cuda.synchronize()
        assert np.array_equal(cost.cpu().numpy().astype(np.float64), want_c)
        assert np.array_equal(end.cpu().numpy(), want_e)
    plan.close()
    ref.close()


LENGTHS = [1, 2, 3, 5, 7, 31, 32, 33, 48, 63, 64, 65, 100, 127, 128, 129, 200, 225, 255, 256, 257,
           400, 512, 513, 777, 1000, 1023, 1024, 1025, 1500, 2000, 2048, 2049]


@pytest.mark.parametrize("dt", ["i16", "f32"])
@pytest.mark.parametrize("n", [1, 3, 4, 5, 63, 255, 257, 1023, 5001])
def test_every_lane_split(dev, n, dt):
    rng = np.random.default_rng(n)
    note(f"rows n={n} {dt}, {len(LENGTHS)} lengths from 1 to 2,049")
    check_batch(dev, values(rng, n, dt), [values(rng, m, dt) for m in LENGTHS], dt)


@pytest.mark.parametrize("dt", ["i16", "f32"])
@pytest.mark.parametrize("nq,lo,hi,n", [(1, 250, 250, 59_796), (3, 1, 40, 30_000),
                                        (40, 20, 300, 59_796), (300, 60, 500, 20_011),
                                        (5, 1500, 2048, 40_000)])
def test_segments_settle(dev, nq, lo, hi, n, dt):
    rng = np.random.default_rng(nq)
    g = synth.make_genome(n // 2 + 5, n)
    z, codes, _ = oracle.prepare_reference(g, synth.make_level_table(), 6)
    rd = synth.simulate_reads(g, synth.make_level_table(), rng.integers(lo, hi + 1, size=nq), 0.5,
                              n + nq)
    qz, qc, _ = oracle.prepare_queries(rd.values, rd.offsets)
    q = qc if dt == "i16" else qz
    note(f"rows {nq} reads of {lo}-{hi} vs {codes.size} {dt}")
    check_batch(dev, codes if dt == "i16" else z,
                [q[rd.offsets[i]:rd.offsets[i + 1]] for i in range(nq)], dt)


def flat_references(rng, n, dt):
    """References with stretches without variation at the queries' own values."""
    half = values(rng, n, dt, 500)
    half[n // 3:2 * n // 3] = 0
    ties = rng.integers(0, 3, size=n).astype(half.dtype)
    steps = np.repeat(rng.integers(0, 9, size=n // 4000 + 1), 4000)[:n].astype(half.dtype)
    return {"constant": np.zeros(n, half.dtype), "flat third": half, "ties": ties,
            "steps": steps}


@pytest.mark.parametrize("dt", ["i16", "f32"])
@pytest.mark.parametrize("kind", ["constant", "flat third", "ties", "steps"])
def test_segments_that_do_not_settle(dev, kind, dt):
    rng = np.random.default_rng(5)
    ref = flat_references(rng, 40_001, dt)[kind]
    reads = [rng.integers(0, 9, size=m).astype(ref.dtype) for m in (1, 30, 250, 250, 600)]
    note(f"rows {kind} reference {dt}")
    check_batch(dev, ref, reads, dt)


@pytest.mark.parametrize("kind", ["random", "constant", "flat third", "ties", "steps"])
@pytest.mark.parametrize("dt", ["i16", "f32"])
def test_chunks(dev, dt, kind):
    rng = np.random.default_rng(8)
    n = 30_003
    ref_np = values(rng, n, dt) if kind == "random" else flat_references(rng, n, dt)[kind]
    small = kind != "random"
    plans = [[400, 400, 30], [1, 2, 65], [250, 64, 1], [2000, 100, 3], [2100, 33, 300], [5, 7, 9]]
    reads = [(rng.integers(0, 9, size=sum(p)).astype(ref_np.dtype) if small
              else values(rng, sum(p), dt)) for p in plans]
    ref = sd.Reference(torch.from_numpy(ref_np).to(dev))
    streams = [sd.Stream(ref) for _ in plans]
    for k in range(3):
        cuts = [(sum(p[:k]), sum(p[:k + 1])) for p in plans]
        q, offs = synth.csr([r[a:b] for r, (a, b) in zip(reads, cuts)])
        note(f"rows chunk {k} vs {kind} {dt}")
        cost, end = sd.stream_extend(streams, torch.from_numpy(q.astype(ref_np.dtype)).to(dev),
                                     offs)
        torch.cuda.synchronize()
        for i, (a, b) in enumerate(cuts):
            fn = oracle.sdtw_i64 if dt == "i16" else oracle.sdtw_f32
            wc, we, lr = fn(reads[i][:b], ref_np, lastrow=True)
            assert (float(cost[i].item()), int(end[i].item())) == (float(wc), we), (i, k)
            row = streams[i].copy_row().cpu().numpy()
            assert np.array_equal(row.astype(np.float64), lr.astype(np.float64)), (i, k)
    for s in streams:
        s.close()
    ref.close()


@pytest.mark.parametrize("kind", ["constant", "flat third", "steps"])
def test_one_read_on_a_long_flat_reference(dev, kind):
    # long enough that the row scan takes over where most segments stay
    # unsettled (and does nothing where few do), also extending a row
    rng = np.random.default_rng(12)
    ref_np = flat_references(rng, 1_100_003, "i16")[kind]
    q = rng.integers(0, 9, size=90).astype(np.int16)
    ref = sd.Reference(torch.from_numpy(ref_np).to(dev))
    note(f"rows one read vs 1,100,003 columns, {kind}")
    want = oracle.sdtw_i64(q, ref_np, lastrow=True)
    qd = torch.from_numpy(q).to(dev)
    c, e = sd.align_one_wide(ref, qd)
    cost = torch.full((1,), -7, dtype=torch.int32, device=dev)
    end = torch.full((1,), -7, dtype=torch.int32, device=dev)
    sd.align_one_wide_noalloc(ref, qd, cost, end)
    s = sd.Stream(ref)
    sd.stream_extend_wide(s, qd[:40].contiguous())
    c2, e2 = sd.stream_extend_wide(s, qd[40:].contiguous())
    for got in ((c, e), (cost, end), (c2, e2)):
        assert (int(got[0].item()), int(got[1].item())) == want[:2]
    assert np.array_equal(s.copy_row().cpu().numpy().astype(np.int64), want[2])
    s.close()
    ref.close()


def test_one_read_and_one_chunk(dev):
    """A read and its chunks alone over the device, mixed with the shapes that
    run the other kernels on the same resident row."""
    rng = np.random.default_rng(9)
    g = synth.make_genome(40_000, 3)
    _, ref_np, _ = oracle.prepare_reference(g, synth.make_level_table(), 6)
    rd = synth.simulate_reads(g, synth.make_level_table(), [1400], 1.0, 4)
    _, q, _ = oracle.prepare_queries(rd.values, rd.offsets)
    ref = sd.Reference(torch.from_numpy(ref_np).to(dev))
    s = sd.Stream(ref)
    at = 0
    for m, how in ((400, "auto"), (100, "cols"), (300, "auto"), (50, "batch"), (64, "shape"),
                   (1, "auto"), (300, "auto"), (185, "batch")):
        chunk = torch.from_numpy(q[at:at + m].copy()).to(dev)
        note(f"rows chunk of {m} at {at} ({how})")
        at += m
        if how in ("auto", "cols"):
            c, e = sd.stream_extend_wide(s, chunk, cols=8 if how == "cols" else 0)
        else:
            if how == "shape":
                sd.set_stream_config(16, 1, ref=ref)
            c, e = sd.stream_extend([s], chunk, np.array([0, m], np.int64))
            sd.set_stream_config(0, 0, ref=ref)
        torch.cuda.synchronize()
        assert (int(c.item()), int(e.item())) == oracle.sdtw_i64(q[:at], ref_np), at
    s.close()
    for m in (1, 30, 250, 1000, 1400):
        c, e = sd.align_one_wide(ref, torch.from_numpy(q[:m].copy()).to(dev))
        assert (int(c.item()), int(e.item())) == oracle.sdtw_i64(q[:m], ref_np), m
    ref.close()
