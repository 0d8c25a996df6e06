"""Track lists whose host arrays do not fit memory: the entry points return
IT_EINVAL, and nothing leaves the C ABI as an exception (which would end the
process).  In a child process whose address space is limited once the tracks
are there; no device is touched before the arrays are made."""
import subprocess
import sys

import pytest

CHILD = r"""
import ctypes, resource, sys
import numpy as np
from paper_1610_06749_amd import binding as B
import workloads as W
L = B.lib()
n = 3_000_000
ch = W.chamber(16, 12, 10, 5e-4, 5e-3, 100.0, reaction_limit=0.0 if sys.argv[1] != "dt" else 0.5)
tr, ptr = B._tracks(np.tile([1.0, 1e-3, 1e-3, 1e-3, 0.0, 0.0, 0.0], (n, 1)))
c = B._chamber(ch)
res = B.it_result()
offs = np.array([0, n], dtype=np.int64)
ws, big, out = ctypes.c_void_p(4096), 1 << 50, ctypes.c_double()
calls = dict(
    solve=lambda: L.it_solve(ctypes.byref(c), ptr, n, None, ws, big, None, None, None, None, ctypes.byref(res)),
    batch=lambda: L.it_solve_batch(ctypes.byref(c), offs.ctypes.data, tr.ctypes.data, 1, None, ws, big, None,
                                   ctypes.byref(res)),
    dt=lambda: L.it_dt(ctypes.byref(c), ptr, n, ctypes.byref(out)))
L.it_solve(None, None, 0, None, None, 0, None, None, None, None, ctypes.byref(res))  # the runtime is up
pages = int(open("/proc/self/statm").read().split()[0])
limit = pages * resource.getpagesize() + (8 << 20)
resource.setrlimit(resource.RLIMIT_AS, (limit, limit))
rc = calls[sys.argv[1]]()
print("returned", rc, B.IT_EINVAL, flush=True)
"""


@pytest.mark.parametrize("call", ["solve", "batch", "dt"])
def test_tracks_that_do_not_fit_host_memory(call):
    r = subprocess.run([sys.executable, "-c", CHILD, call], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-500:]
    word, rc, want = r.stdout.split()[-3:]
    assert word == "returned" and rc == want
