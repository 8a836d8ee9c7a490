"""References without variation: a column segment's left column depends on
everything to its left there, so the calls that cut the reference into
segments leave it to the kernels that do not.  Results equal the oracle, and a
call without a launch shape takes no longer than one that names the shape or
columns per thread of those kernels (half as long again for the noise of one
measurement; segments that one wave walks took 1.3 to 33 times as long).
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


def fastest(call):
    best = float("inf")
    for _ in range(4):
        torch.cuda.synchronize()
        e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        e0.record()
        out = call()
        e1.record()
        torch.cuda.synchronize()
        best = min(best, e0.elapsed_time(e1))
    return best, out


@pytest.mark.parametrize("dt", ["i16", "f32"])
@pytest.mark.parametrize("n", [59_796, 500_000])
def test_constant_reference(n, dt):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(n)
    ref_np = np.full(n, 7, np.int16 if dt == "i16" else np.float32)
    ref = sd.Reference(torch.from_numpy(ref_np).to(dev))
    fn, code = (oracle.sdtw_i64, sd.I16) if dt == "i16" else (oracle.sdtw_f32, sd.F32)
    short = ref_np[:2000]  # (every column of a row is the same after a few)

    def values(m):
        v = rng.integers(-200, 200, m)
        return v.astype(np.int16) if dt == "i16" else (v / 64).astype(np.float32)

    # batches, small and filling the device
    for nq in (8, 1024):
        q, offs = synth.csr([values(250) for _ in range(nq)])
        q = q.astype(ref_np.dtype)
        qd = torch.from_numpy(q).to(dev)
        plan, shaped = sd.Plan(offs, code), sd.Plan(offs, code)
        c = shaped.config
        shaped.set_config(c["strip"], c["chains"], c["waves_per_cu"], c["bands"])
        want = fastest(lambda: sd.align_batch(ref, shaped, qd))[0]
        got, (cost, end) = fastest(lambda: sd.align_batch(ref, plan, qd))
        note(f"flat n={n} {dt} batch of {nq}: {got:.3f} ms, {want:.3f} with the shape set")
        for i in (0, nq - 1):
            assert (float(cost[i].item()), int(end[i].item())) == \
                tuple(map(float, fn(q[250 * i:250 * i + 250], short)))
        plan.close()
        shaped.close()
        assert got < 1.5 * want

    # chunks
    ns = 64
    q, offs = synth.csr([values(400) for _ in range(ns)])
    q = q.astype(ref_np.dtype)
    qd = torch.from_numpy(q).to(dev)
    streams = [sd.Stream(ref) for _ in range(ns)]
    sd.set_stream_config(16 if n < 1 << 20 else 32, 4, ref=ref)
    want = fastest(lambda: sd.stream_extend(streams, qd, offs))[0]
    sd.set_stream_config(0, 0, ref=ref)
    got = fastest(lambda: sd.stream_extend(streams, qd, offs))[0]
    note(f"flat n={n} {dt} {ns} chunks: {got:.3f} ms, {want:.3f} with the shape set")
    assert got < 1.5 * want
    for s in streams:
        s.close()

    # one read and one chunk over the whole device
    if dt == "i16":
        v = values(250)
        qd = torch.from_numpy(v).to(dev)
        want = min(fastest(lambda: sd.align_one_wide(ref, qd, cols=c))[0] for c in (8, 16, 32))
        got, (cost, end) = fastest(lambda: sd.align_one_wide(ref, qd))
        note(f"flat n={n} one read: {got:.3f} ms, {want:.3f} by row scans")
        assert (int(cost.item()), int(end.item())) == fn(v, short)
        assert got < 1.5 * want
        s = sd.Stream(ref)
        want = min(fastest(lambda: sd.stream_extend_wide(s, qd, cols=c))[0] for c in (8, 16, 32))
        got = fastest(lambda: sd.stream_extend_wide(s, qd))[0]
        note(f"flat n={n} one chunk: {got:.3f} ms, {want:.3f} by row scans")
        assert got < 1.5 * want
        s.close()
    ref.close()


@pytest.mark.parametrize("dt", ["i16", "f32"])
def test_flat_share_decides_alone(dt):
    """Around the share where the route changes, and runs off the 64-column
    grid: the same results."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(4)
    n = 12 * 1024
    for at, run in ((0, 1024), (64, 1088), (33, 1150), (n - 1090, 1090), (5, 63)):
        v = rng.integers(-3000, 3000, n)
        v[at:at + run] = 11
        ref_np = v.astype(np.int16) if dt == "i16" else (v / 64).astype(np.float32)
        reads = [rng.integers(-3000, 3000, m).astype(np.int16) for m in (1, 70, 300)]
        if dt == "f32":
            reads = [(r / 64).astype(np.float32) for r in reads]
        note(f"flat run of {run} at {at} of {n} {dt}")
        q, offs = synth.csr(reads)
        q = q.astype(ref_np.dtype)
        kind, code = (oracle.I64, sd.I16) if dt == "i16" else (oracle.F32, sd.F32)
        wc, we, _ = oracle.batch(kind, q, offs, ref_np)
        ref = sd.Reference(torch.from_numpy(ref_np).to(dev))
        plan = sd.Plan(offs, code)
        cost, end = sd.align_batch(ref, plan, torch.from_numpy(q).to(dev))
        streams = [sd.Stream(ref) for _ in reads]
        sc, se = sd.stream_extend(streams, torch.from_numpy(q).to(dev), offs)
        torch.cuda.synchronize()
        for c, e in ((cost, end), (sc, se)):
            assert np.array_equal(c.cpu().numpy().astype(np.float64), wc)
            assert np.array_equal(e.cpu().numpy(), we)
        for s in streams:
            s.close()
        plan.close()
        ref.close()


def test_one_read_where_many_segments_stay_unsettled():
    """Values that differ from column to column by next to nothing are no run of
    equal values: on a long reference the row scan takes over on the device."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(3)
    n = 1_100_003
    ref_np = (np.arange(n) % 2).astype(np.int16)
    q = rng.integers(-300, 300, 90).astype(np.int16)
    ref = sd.Reference(torch.from_numpy(ref_np).to(dev))
    qd = torch.from_numpy(q).to(dev)
    note("alternating reference, one read and two chunks")
    s = sd.Stream(ref)
    for _ in range(2):
        cost, end = sd.align_one_wide(ref, qd)
        assert (int(cost.item()), int(end.item())) == oracle.sdtw_i64(q, ref_np)
    sd.stream_extend_wide(s, qd[:40].contiguous())
    cost, end = sd.stream_extend_wide(s, qd[40:].contiguous())
    wc, we, lr = oracle.sdtw_i64(q, ref_np, lastrow=True)
    assert (int(cost.item()), int(end.item())) == (wc, we)
    assert np.array_equal(s.copy_row().cpu().numpy().astype(np.int64), lr)
    s.close()
    ref.close()
