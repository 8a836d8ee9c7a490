"""A call that runs out of host memory returns SDTW_ENOMEM through the C ABI
instead of ending the process (no GPU needed: the plan's host side comes first)."""
import os
import subprocess
import sys
import textwrap

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CODE = textwrap.dedent("""
    import ctypes as C, resource, sys
    import numpy as np
    sys.path.insert(0, %r)
    import paper_2211_07340_amd as sd
    lib = sd.load_library()
    nq = 20_000_000
    offs = np.arange(nq + 1, dtype=np.int64)
    out = C.c_void_p()
    now = [int(l.split()[1]) << 10 for l in open("/proc/self/status") if l.startswith("VmSize")][0]
    for more in (40, 120, 200, 400):  # MB: short of the first list, the lengths, the layouts
        resource.setrlimit(resource.RLIMIT_AS, (now + (more << 20), resource.RLIM_INFINITY))
        rc = lib.sdtw_plan_create(offs.ctypes.data_as(C.c_void_p), nq, 1, C.byref(out))
        resource.setrlimit(resource.RLIMIT_AS, (resource.RLIM_INFINITY, resource.RLIM_INFINITY))
        print(more, rc, lib.sdtw_last_error().decode(), flush=True)
""") % ROOT


def test_plan_without_host_memory():
    if not os.path.exists(os.path.join(ROOT, "paper_2211_07340_amd", "libsdtw.so")):
        import __graft_entry__
        __graft_entry__.build()
    r = subprocess.run([sys.executable, "-c", CODE], capture_output=True, text=True, timeout=200)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr[-500:])
    lines = r.stdout.splitlines()
    assert len(lines) == 4
    for line in lines:
        assert line.split()[1] == "2" and line.endswith("host allocation"), line
