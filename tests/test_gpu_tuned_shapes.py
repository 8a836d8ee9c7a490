"""Tuned launch shapes of plans with reads over 2,048 rows: the timing loop runs
for them, what it finds is applied to plans of the same class, and tuning a plan
that has nothing to tune leaves it alone, also in the file."""
import os
import subprocess
import sys
import textwrap

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
sd = pytest.importorskip("paper_2211_07340_amd")

N = 20_000
LONG = [2100] * 4 + [2000] * 8   # median 2,000, longest in the bucket of 2,048
SHORT = [2048] * 4 + [2000] * 8

CODE = textwrap.dedent("""
    import sys, numpy as np, torch
    sys.path.insert(0, %r)
    import paper_2211_07340_amd as sd
    from tests.test_gpu_tuned_shapes import LONG, SHORT, batch, reference
    ref = sd.Reference(torch.from_numpy(reference()).cuda())
    def plan(lens):
        q, offs = batch(lens)
        return sd.Plan(offs, sd.I16), torch.from_numpy(q).cuda()
    if sys.argv[1] == "long":
        p, q = plan(LONG)
        print(sd.autotune(ref, p, q, max_columns=8192))
    else:
        p, q = plan(SHORT)
        sd.autotune(ref, p, q)
        p, q = plan(LONG)
        print(sd.use_tuned(ref, p), p.config)
    torch.cuda.synchronize()
""")


def reference():
    return np.random.default_rng(1).integers(-3000, 3000, N).astype(np.int16)


def batch(lens):
    rng = np.random.default_rng(2)
    return synth.csr([rng.integers(-3000, 3000, m).astype(np.int16) for m in lens])


def run(what, path):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    print(f"tuned shapes: {what}", flush=True)
    sys.stdout.flush()
    r = subprocess.run([sys.executable, "-c", CODE % root, what], capture_output=True, text=True,
                       env=dict(os.environ, SDTW_TUNE_CACHE=str(path)), timeout=200, cwd=root)
    assert r.returncode == 0, r.stderr[-2000:]
    return r.stdout.strip().splitlines()[-1]


def test_shape_of_long_reads_stays(tmp_path):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    path = tmp_path / "tune.txt"
    run("long", path)
    lines = path.read_text().splitlines()
    assert len(lines) == 1
    # another shape than the timed and the default one stands in for it
    key = lines[0].split()[:7]
    given = " ".join(key + ["16", "1", "1", "3", "0"])
    path.write_text(given + "\n")
    out = run("short", path)
    assert out == "True " + str({"strip": 16, "chains": 1, "bands": 1, "waves_per_cu": 3,
                                 "band_rows": 0})
    assert given in path.read_text().splitlines()


def test_tuned_mixed_batch_equals_the_oracle():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    lens = [2049, 2100, 3000, 70, 1, 300, 2048]
    q, offs = batch(lens)
    ref_np = reference()
    want_c, want_e, _ = oracle.batch(oracle.I64, q, offs, ref_np)
    ref = sd.Reference(torch.from_numpy(ref_np).to(dev))
    plan = sd.Plan(offs, sd.I16)
    qd = torch.from_numpy(q).to(dev)
    print("autotune of reads of 1 to 3,000 rows", flush=True)
    sys.stdout.flush()
    for _ in range(2):  # as created, then tuned
        cost, end = sd.align_batch(ref, plan, qd)
        torch.cuda.synchronize()
        assert np.array_equal(cost.cpu().numpy(), want_c) and \
            np.array_equal(end.cpu().numpy(), want_e)
        sd.autotune(ref, plan, qd, max_columns=8192)
    other = sd.Plan(offs, sd.I16)
    other.set_config(strip=8, chains=1, bands=1, waves_per_cu=2)
    assert other.config != plan.config
    assert sd.use_tuned(ref, other) and other.config == plan.config
    plan.close()
    other.close()
    ref.close()
