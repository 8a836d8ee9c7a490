"""Device memory that chunk calls hold: a large batch after a small one takes no
more (growing a call's scratch would wait for all work on the device, in the
middle of serving)."""
import sys

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
sd = pytest.importorskip("paper_2211_07340_amd")


def test_scratch_does_not_grow():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(2)
    small = rng.integers(-3000, 3000, 50_000).astype(np.int16)
    large = rng.integers(-3000, 3000, 2_000_003).astype(np.int16)
    q = rng.integers(-3000, 3000, 700 * 100).astype(np.int16)
    qd = torch.from_numpy(q).to(dev)
    offs = np.arange(701, dtype=np.int64) * 100
    refs = [sd.Reference(torch.from_numpy(r).to(dev)) for r in (small, large)]
    few = [sd.Stream(refs[0]) for _ in range(8)]
    many = [sd.Stream(refs[1]) for _ in range(700)]
    cost = torch.empty(700, dtype=torch.int32, device=dev)
    end = torch.empty(700, dtype=torch.int32, device=dev)
    sd.stream_extend(few, qd, offs[:9], cost[:8], end[:8])
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    print("700 chunks x 2,000,003 columns after 8 x 50,000", flush=True)
    sys.stdout.flush()
    sd.stream_extend(many, qd, offs, cost, end)
    torch.cuda.synchronize()
    after = torch.cuda.mem_get_info()[0]
    assert before - after < 1 << 20
    for i in (0, 699):
        assert (int(cost[i].item()), int(end[i].item())) == \
            oracle.sdtw_i64(q[100 * i:100 * i + 100], large)
    for s in few + many:
        s.close()
    for r in refs:
        r.close()
    sd.row_pool_trim()
