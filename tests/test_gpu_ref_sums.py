"""Reference statistics (sums in index order, found in parallel): z bits, codes
and saturation counts equal the oracle's plain loop at tile edges, for level
tables whose sums cross binades often, tie in rounding, are negative, zero,
huge, tiny or not finite.
"""
import sys

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
sd = pytest.importorskip("paper_2211_07340_amd")


def tables(kind, rng):
    n = 4 ** 3
    t = {
        "currents": rng.normal(90, 12, n),
        "signed": rng.normal(0, 12, n),
        "mostly zero": np.where(rng.random(n) < 0.9, 0.0, 1.0),
        "wide": 10.0 ** rng.uniform(-12, 12, n),           # terms far below an ulp of the sum
        "halves": rng.integers(1, 5, n) * 0.5 + 2.0 ** 23,  # many exact ties
        "large": 10.0 ** rng.uniform(30, 38, n),
        "tiny": 10.0 ** rng.uniform(-44, -38, n),
        "equal": np.full(n, 77.25),
        "nan": np.where(np.arange(n) == 5, np.nan, 80.0),
        "inf": np.where(np.arange(n) == 5, np.inf, 80.0),
    }[kind]
    return t.astype(np.float32)


@pytest.mark.parametrize("kind", ["currents", "signed", "mostly zero", "wide", "halves", "large",
                                  "tiny", "equal", "nan", "inf"])
def test_sums_in_index_order(kind):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(7)
    table = tables(kind, rng)
    for L in (3, 4, 10, 514, 515, 1026, 2050, 30_003, 70_001):
        g = synth.make_genome(L, L)
        print(f"reference sums {kind} L={L}", flush=True)
        sys.stdout.flush()
        z, codes, nsat = sd.prepare_reference(torch.from_numpy(g).to(dev),
                                              torch.from_numpy(table).to(dev), 3, 64.0)
        torch.cuda.synchronize()
        with np.errstate(all="ignore"):
            wz, wc, ws = oracle.prepare_reference(g, table, 3)
        assert np.array_equal(z.cpu().numpy().view(np.uint32), wz.view(np.uint32)) or (
            kind in ("nan", "inf") and np.array_equal(z.cpu().numpy(), wz, equal_nan=True)), L
        if kind not in ("nan", "inf"):
            assert np.array_equal(codes.cpu().numpy(), wc), L
            assert int(nsat.item()) == int(ws), L
