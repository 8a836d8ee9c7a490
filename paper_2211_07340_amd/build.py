"""Build the HIP library ``libsdtw.so`` for gfx950 with hipcc (in-tree)."""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsdtw.so")
SOURCES = ["rows_i16.hip", "rows_f32.hip", "rows_i16_stream.hip", "rows_f32_stream.hip",
           "align.hip", "api.hip", "prep.hip", "scores.hip", "wide.hip", "events.hip"]
ARCH = os.environ.get("SDTW_OFFLOAD_ARCH", "gfx950")

FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "-shared",
    f"--offload-arch={ARCH}",
    # exact IEEE arithmetic: no contraction, no fast-math, fp32 denormals kept
    "-ffp-contract=off", "-fno-fast-math",
    # no packed-fp32 instructions anywhere
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-result",
]


PROBE_LIB = os.path.join(HERE, "libsdtw_probe.so")
PROBE_SOURCES = ["probe_issue.hip"]


def build_probe(verbose: bool = False) -> str:
    """The VALU issue-rate probe (libsdtw_probe.so, measurement tooling)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *FLAGS, "-o", PROBE_LIB + ".tmp",
           *[os.path.join(CSRC, s) for s in PROBE_SOURCES]]
    proc = subprocess.run(cmd, capture_output=True, text=True, cwd=HERE)
    out = "\n".join(l for l in (proc.stdout + proc.stderr).splitlines()
                    if "packed-fp32-ops" not in l)
    if proc.returncode != 0:
        raise RuntimeError(f"hipcc failed ({proc.returncode}):\n{out}")
    if verbose and out.strip():
        print(out, file=sys.stderr)
    os.replace(PROBE_LIB + ".tmp", PROBE_LIB)
    return PROBE_LIB


def _compile(src: str, obj: str, save_temps: str | None):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *[f for f in FLAGS if f != "-shared"], "-c", "-o", obj,
           os.path.join(CSRC, src)]
    if save_temps:
        cmd.insert(1, "-save-temps=obj")
    return subprocess.run(cmd, capture_output=True, text=True, cwd=HERE)


def build(verbose: bool = False, save_temps: str | None = None) -> str:
    """Compile the sources side by side and link them."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    workers = int(os.environ.get("MAX_JOBS", "0")) or min(len(SOURCES), os.cpu_count() or 1)
    with tempfile.TemporaryDirectory() as tmp, ThreadPoolExecutor(workers) as pool:
        into = save_temps or tmp
        os.makedirs(into, exist_ok=True)
        objs = [os.path.join(into, s + ".o") for s in SOURCES]
        done = list(pool.map(_compile, SOURCES, objs, [save_temps] * len(SOURCES)))
        if all(p.returncode == 0 for p in done):
            done.append(subprocess.run([hipcc, *FLAGS, "-o", LIB + ".tmp", *objs],
                                       capture_output=True, text=True, cwd=HERE))
    out = "\n".join(l for p in done for l in (p.stdout + p.stderr).splitlines()
                    if "packed-fp32-ops" not in l)
    bad = [p.returncode for p in done if p.returncode != 0]
    if bad:
        raise RuntimeError(f"hipcc failed ({bad[0]}):\n{out}")
    if verbose and out.strip():
        print(out, file=sys.stderr)
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
    print(build_probe(verbose=True))
