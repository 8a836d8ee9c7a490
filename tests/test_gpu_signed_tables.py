"""Reference statistics for level tables with negative values (tables in
normalised units): no map of sums exists for a run with a negative term, so
most of the first sum is added up term by term, as both sums are for small
genomes.  Same bits as the oracle, and no slower than the plain loop of one wave,
which prepares the same signal as one read's events.
"""
import sys

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
sd = pytest.importorskip("paper_2211_07340_amd")


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


def prepare(bases, share):
    """A level table of which `share` is negative: device inputs and the oracle's outputs."""
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(int(1e4 * share) + bases)
    table = np.abs(rng.normal(0.0, 1.0, 4 ** 6)).astype(np.float32)
    table[rng.random(table.size) < share] *= -1
    g = synth.make_genome(bases, 7)
    return (torch.from_numpy(g).to(dev), torch.from_numpy(table).to(dev),
            oracle.prepare_reference(g, table, 6))


def check(got, want):
    assert np.array_equal(got[0].cpu().numpy().view(np.uint32), want[0].view(np.uint32))
    assert np.array_equal(got[1].cpu().numpy(), want[1]) and int(got[2].item()) == int(want[2])


# share of negative levels: none of a tile's 64 runs of 16, a few, most, all
@pytest.mark.parametrize("share", [0.0001, 0.004, 0.03, 0.5, 1.0])
@pytest.mark.parametrize("bases", [29_903, 300_001])
def test_signed_levels(bases, share):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g, table, want = prepare(bases, share)
    took, got = fastest(lambda: sd.prepare_reference(g, table, 6, 64.0))
    check(got, want)
    raw = torch.rand(got[0].numel(), device="cuda:0")
    offs = torch.tensor([0, raw.numel()], dtype=torch.int64, device="cuda:0")
    plain, _ = fastest(lambda: sd.prepare_queries(raw, offs, 64.0))
    print(f"signed levels {share} of {bases} bases: {took:.3f} ms, plain loop {plain:.3f}",
          flush=True)
    sys.stdout.flush()
    assert took < plain


# 2, 32 (two runs of 16), 34, 1,022, 1,024, 1,026 values and the most that one
# wave adds up in one launch (5,120) and two more
@pytest.mark.parametrize("share", [0.0, 0.03, 1.0])
@pytest.mark.parametrize("bases", [6, 21, 22, 516, 517, 518, 2565, 2566])
def test_small_genomes(bases, share):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g, table, want = prepare(bases, share)
    print(f"small genome of {bases} bases, {share} negative", flush=True)
    sys.stdout.flush()
    check(sd.prepare_reference(g, table, 6, 64.0), want)
