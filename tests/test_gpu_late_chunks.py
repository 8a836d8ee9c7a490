"""Short chunks late in the course of an on-target read: the resident row's
minimum lies far below its other costs there, and a column segment's left
column depends on as many columns as a path takes to climb between the two.
Extensions equal the oracle bit for bit and are not slower by more than that:
a chunk's halo grows from 100 to at most 2,200 columns (3,600 rows held), a
fraction of the 59,796-column sweep, so four times the time of a chunk of the
same rows early in the read leaves room (a reference walked by one wave per
read instead took ten times as long).
"""
import sys

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
sd = pytest.importorskip("paper_2211_07340_amd")

EARLY, CALLS = 400, 6


def note(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("dt", ["i16", "f32"])
@pytest.mark.parametrize("held,m,ns", [(2000, 40, 8), (3600, 64, 3), (3600, 20, 1)])
def test_late_chunks(held, m, ns, dt):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    table = synth.make_level_table()
    g = synth.make_genome(29_903, 17)
    z, codes, _ = oracle.prepare_reference(g, table, 6)
    ref_np = codes if dt == "i16" else z
    L = held + CALLS * m
    rd = synth.simulate_reads(g, table, [L] * ns, 1.0, 23, noise_sd=1.2)
    qz, qc, _ = oracle.prepare_queries(rd.values, rd.offsets)
    q = (qc if dt == "i16" else qz).reshape(ns, L)
    ref = sd.Reference(torch.from_numpy(ref_np).to(dev))
    streams = [sd.Stream(ref) for _ in range(ns)]
    wide = sd.Stream(ref)

    def extend(to, a, b):
        chunk = torch.from_numpy(np.ascontiguousarray(q[:len(to), a:b]).reshape(-1)).to(dev)
        return chunk, np.arange(len(to) + 1, dtype=np.int64) * (b - a)

    def grow(to, upto):
        at = 0
        while at < upto:
            step = min(400, upto - at)
            sd.stream_extend(to, *extend(to, at, at + step))
            at += step

    def time_calls(at, whole):
        to = [wide] if whole else streams
        best = float("inf")
        for k in range(CALLS):
            chunk, offs = extend(to, at, at + m)
            at += m
            torch.cuda.synchronize()
            e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            e0.record()
            out = sd.stream_extend_wide(wide, chunk) if whole else sd.stream_extend(to, chunk, offs)
            e1.record()
            torch.cuda.synchronize()
            best = min(best, e0.elapsed_time(e1))
        return best, out

    ways = [False] + ([True] if dt == "i16" and L <= 4096 else [])
    for whole in ways:
        note(f"late chunks {dt}: {ns} reads, {held} rows held, chunks of {m}, whole={whole}")
        to = [wide] if whole else streams
        grow(to, EARLY)
        early, _ = time_calls(EARLY, whole)
        at = EARLY + CALLS * m
        while at < held:
            step = min(400, held - at)
            sd.stream_extend(to, *extend(to, at, at + step))
            at += step
        late, (cost, end) = time_calls(held, whole)
        note(f"  early {early:.3f} ms, late {late:.3f} ms")
        fn = oracle.sdtw_i64 if dt == "i16" else oracle.sdtw_f32
        for i, s in enumerate(to):
            wc, we, lr = fn(q[i], ref_np, lastrow=True)
            assert (float(cost[i].item()), int(end[i].item())) == (float(wc), we), i
            assert np.array_equal(s.copy_row().cpu().numpy().astype(np.float64),
                                  lr.astype(np.float64)), i
        assert late < 4 * early
    for s in streams + [wide]:
        s.close()
    ref.close()
