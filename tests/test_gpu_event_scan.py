"""Event detection by a wave that starts the detectors blank in every lane
and mends: against the oracle where lanes disagree with their neighbours (long
stretches in which the state stays what it was, candidates that stay open over
one or several blocks of 1,024 positions) and at the blocks' and lanes' edges.
"""
import sys

import numpy as np
import pytest

from oracle import events as oev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
sd = pytest.importorskip("paper_2211_07340_amd")


def signals():
    rng = np.random.default_rng(3)
    s = {}
    for L in (0, 1, 5, 6, 11, 12, 13, 17, 1023, 1024, 1025, 1029, 1030, 2047, 2050, 3100):
        lv = np.repeat(rng.normal(90, 12, L // 4 + 1), rng.integers(4, 14, L // 4 + 1))[:L]
        s[f"levels {L}"] = lv + rng.normal(0, 1.5, lv.size)
    s["flat"] = np.full(2500, 80.0)
    s["ramp"] = np.linspace(60, 120, 3000)
    s["slow wave"] = 90 + 20 * np.sin(np.arange(4000) / 700.0)
    s["one step"] = np.where(np.arange(3000) < 1500, 80.0, 95.0)
    # steps without noise, so far apart that candidates stay open for blocks
    s["rare steps"] = 80.0 + 10.0 * (np.arange(6000) // 1300)
    s["step then flat"] = np.concatenate([rng.normal(90, 5, 40), np.full(4200, 90.0),
                                          rng.normal(90, 12, 300)])
    s["bursts"] = np.concatenate([np.full(1500, 75.0), rng.normal(90, 12, 100),
                                  np.full(1500, 99.0), rng.normal(90, 12, 100)] * 2)
    # one candidate over three blocks: t rises a little for ever
    s["creeping"] = 90 + np.cumsum(np.linspace(0, 0.02, 3500)) + 0.01 * (np.arange(3500) % 3)
    x = rng.normal(90, 5, 2100)
    x[1030] = np.inf
    s["inf"] = x
    x = rng.normal(90, 5, 2100)
    x[700] = np.nan
    s["nan"] = x
    s["large"] = rng.normal(0, 1, 1500) * 1e30
    s["tiny"] = rng.normal(0, 1, 1500) * 1e-42
    return {k: np.asarray(v, np.float32) for k, v in s.items()}


def tstat_fmax(x, w):
    """The oracle's t statistic with C's fmax for the denominator's floor: the
    same for finite samples; a NaN deviation counts as 0 in the library, while
    Python's max would keep it."""
    v = np.asarray(x, np.float64)
    t = np.zeros(v.size)
    for i in range(w, v.size - w + 1):
        s = [0.0, 0.0]
        q = [0.0, 0.0]
        for side, at in ((0, i - w), (1, i)):
            for k in range(w):
                s[side] = s[side] + v[at + k]
            s[side] = s[side] / w
            for k in range(w):
                q[side] = q[side] + (v[at + k] - s[side]) * (v[at + k] - s[side])
            q[side] = q[side] / w
        t[i] = abs(s[1] - s[0]) / np.fmax(np.sqrt((q[0] + q[1]) / w), oev.DEN_FLOOR)
    return t


def events_of(x):
    v = np.asarray(x, np.float64)
    if np.isfinite(v).all():
        return oev.events(x)
    cuts = [0] + [b for b in oev.peaks(tstat_fmax(x, 3), tstat_fmax(x, 6))
                  if 0 < b < v.size] + [v.size]
    out = []
    for a, b in zip(cuts[:-1], cuts[1:]):
        s = 0.0
        for k in range(a, b):
            s = s + v[k]
        out.append(s / (b - a))
    return np.asarray(out, np.float64).astype(np.float32)


@pytest.fixture(scope="module")
def want():
    with np.errstate(all="ignore"):
        x = signals()["levels 1025"]
        assert np.array_equal(tstat_fmax(x, 3), oev.tstat(x, 3))
        return {k: (x, events_of(x)) for k, x in signals().items()}


def same(a, b):
    return np.array_equal(a.view(np.uint32), np.asarray(b, np.float32).view(np.uint32)) or \
        np.array_equal(a, b, equal_nan=True)


@pytest.mark.parametrize("trim,keep", [(0, 900), (3, 40), (50, 4096), (0, 1)])
def test_whole_reads(want, trim, keep):
    dev = torch.device("cuda:0")
    xs = [w[0] for w in want.values()]
    offs = np.concatenate([[0], np.cumsum([x.size for x in xs])]).astype(np.int64)
    print(f"whole reads trim={trim} keep={keep}", flush=True)
    sys.stdout.flush()
    ev, cnt = sd.detect_events(torch.from_numpy(np.concatenate(xs)).to(dev),
                               torch.from_numpy(offs).to(dev), trim, keep)
    torch.cuda.synchronize()
    ev, cnt = ev.cpu().numpy(), cnt.cpu().numpy()
    for r, (name, (x, events)) in enumerate(want.items()):
        e = events[trim:trim + keep]
        assert cnt[r] == e.size, name
        assert same(ev[r, :e.size], e), name
        assert not ev[r, e.size:].any(), name


@pytest.mark.parametrize("sizes", [[1], [7, 300, 2, 1500], [1024], [1029, 1024], [5, 1, 1]])
def test_reads_in_chunks(want, sizes):
    """Delivered events are the whole read's, none that is not final, all that
    are; the state carries every open candidate from call to call."""
    dev = torch.device("cuda:0")
    names = [k for k in want if sizes != [1] or want[k][0].size < 40]
    xs = [want[k][0] for k in names]
    offs = np.concatenate([[0], np.cumsum([x.size for x in xs])]).astype(np.int64)
    raw = torch.from_numpy(np.concatenate(xs)).to(dev)
    n = len(xs)
    states = sd.EventStates(n)
    slots = torch.arange(n, dtype=torch.int32, device=dev)
    states.reset(slots)
    got = [[] for _ in names]
    end, k = 0, 0
    print(f"reads in chunks of {sizes}", flush=True)
    while end < max(x.size for x in xs):
        end += sizes[k % len(sizes)]
        k += 1
        if sizes == [5, 1, 1] and end > 60:
            end += 900
        rg = np.stack([offs[:-1], offs[:-1] + np.minimum(end, np.diff(offs))], 1)
        ev, cnt = states.detect(raw, torch.from_numpy(np.ascontiguousarray(rg)).to(dev), slots, 2,
                                600)
        torch.cuda.synchronize()
        ev, cnt = ev.cpu().numpy(), cnt.cpu().numpy()
        for r in range(n):
            assert cnt[r] >= 0, names[r]
            got[r].append(ev[r, :cnt[r]])
            assert not ev[r, cnt[r]:].any()
    # what a prefix call finds final in one go
    ranges = np.stack([offs[:-1], offs[1:]], 1)
    pe, pc = sd.detect_events_prefix(raw, torch.from_numpy(np.ascontiguousarray(ranges)).to(dev),
                                     torch.full((n,), 2, dtype=torch.int32, device=dev), 2, 4096)
    torch.cuda.synchronize()
    pe, pc = pe.cpu().numpy(), pc.cpu().numpy()
    for r, name in enumerate(names):
        g = np.concatenate(got[r]) if got[r] else np.zeros(0, np.float32)
        events = want[name][1][2:]
        assert same(g, events[:g.size]), name
        assert same(g, pe[r, :pc[r]]), name
