"""Every number of rows per lane of the row-lane kernel against the oracle:
reads whose lanes are all full, all but one, and all one row short, in batches
(four reads to a wave) and in chunks (three), cut into segments and, in the
shortest reference, not.  Bit-exact in both formats.
"""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
sd = pytest.importorskip("paper_2211_07340_amd")


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sd.load_library()
    return torch.device("cuda:0")


def draw(rng, n, dt):
    v = rng.integers(-3000, 3001, size=n)
    return v.astype(np.int16) if dt == "i16" else (v / 64).astype(np.float32)


@pytest.mark.parametrize("dt", ["i16", "f32"])
@pytest.mark.parametrize("n", [61, 6_003])
@pytest.mark.parametrize("rows", list(range(2, 33, 2)))
def test_rows_per_lane(dev, rows, n, dt):
    rng = np.random.default_rng(100 * rows + n)
    print(f"rows per lane {rows} n={n} {dt}", flush=True)
    ref_np = draw(rng, n, dt)
    ref = sd.Reference(torch.from_numpy(ref_np).to(dev))
    fn = oracle.sdtw_i64 if dt == "i16" else oracle.sdtw_f32

    def lengths(lanes):
        return [lanes * rows, lanes * rows - 1, max(lanes * (rows - 1), 1), lanes * rows,
                lanes * rows]

    reads = [draw(rng, m, dt) for m in lengths(16)]
    q, offs = synth.csr(reads)
    plan = sd.Plan(offs, sd.I16 if dt == "i16" else sd.F32)
    cost, end = sd.align_batch(ref, plan, torch.from_numpy(q.astype(ref_np.dtype)).to(dev))
    torch.cuda.synchronize()
    for i, r in enumerate(reads):
        c, e = fn(r, ref_np)[:2]
        assert (float(cost[i].item()), int(end[i].item())) == (float(c), e), i
    plan.close()

    reads = [draw(rng, 2 * m, dt) for m in lengths(21)]
    streams = [sd.Stream(ref) for _ in reads]
    for k in (0, 1):
        q, offs = synth.csr([r[k * r.size // 2:(k + 1) * r.size // 2] for r in reads])
        cost, end = sd.stream_extend(streams, torch.from_numpy(q.astype(ref_np.dtype)).to(dev),
                                     offs)
        torch.cuda.synchronize()
        for i, r in enumerate(reads):
            c, e, last = fn(r[:(k + 1) * r.size // 2], ref_np, lastrow=True)
            assert (float(cost[i].item()), int(end[i].item())) == (float(c), e), (i, k)
            row = streams[i].copy_row().cpu().numpy()
            assert np.array_equal(row.astype(np.float64), last.astype(np.float64)), (i, k)
    for s in streams:
        s.close()
    ref.close()
