"""Host memory running out inside an entry point is an error status, never an
exception or an abort across the C ABI: each call runs in a process of its own
whose address space is limited to little more than it already uses, on stacks
whose analysis needs several times that.  No GPU is needed: every call fails
before its device work."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SCRIPT = r"""
import ctypes as C, resource, sys
import numpy as np
from paper_2607_05818_amd import gen, reff
call, spare = sys.argv[1], int(sys.argv[2]) << 20
rng = np.random.default_rng(0)
nx = ny = 1500
def stack(seed):
    t = np.arange(0, nx * ny, 40)
    return gen.make_desc(2, nx, ny, np.full(2 * ny * (nx - 1), 1.5), np.full(2 * (ny - 1) * nx, 0.5),
                         np.stack([t % nx, t // nx], 1).astype(np.int32), np.ones((len(t), 1)), [[0, 0]])
n = 3 if call in ("selinv_batch", "batch_plans") else 1
descs = [stack(i) for i in range(n)]
structs = (reff.reff_pdn_desc * n)()
keep = []
for i, d in enumerate(descs):
    structs[i], k = reff._desc_struct(d)
    keep.append(k)
out = np.zeros(4)
node = np.zeros(4, dtype=np.int64)
nodes = (C.c_void_p * n)(*[node.ctypes.data] * n)
counts = (C.c_int64 * n)(*[4] * n)
outs = (C.c_void_p * n)(*[out.ctypes.data] * n)
info = reff.reff_selinv_stats()
handle = C.c_void_p()
now = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (now + spare, resource.RLIM_INFINITY))
if call == "selinv_info":
    s = reff._lib.reff_selinv_info(C.byref(structs[0]), C.byref(info))
elif call == "build_pdn":
    s = reff._lib.reff_build_pdn(C.byref(structs[0]), 0, C.byref(handle))
elif call == "selinv_batch":
    s = reff._lib.reff_selinv_batch(structs, n, nodes, counts, outs, None, None)
else:
    s = reff._lib.reff_batch_plans(structs, n, nodes, counts, outs, None, None)
resource.setrlimit(resource.RLIMIT_AS, (resource.RLIM_INFINITY, resource.RLIM_INFINITY))
print("status", s, "handle", handle.value, "out", out.tolist(), reff.reff_last_error())
"""


# with 16 MB to spare no further thread can be had either (a stack is 8 MB, an
# allocation arena 64 MB)
@pytest.mark.parametrize("spare", [16, 96])
@pytest.mark.parametrize("call", ["selinv_info", "build_pdn", "selinv_batch", "batch_plans"])
def test_out_of_host_memory(call, spare):
    r = subprocess.run([sys.executable, "-c", SCRIPT, call, str(spare)], cwd=ROOT, capture_output=True,
                       text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    from paper_2607_05818_amd import reff
    assert f"status {reff.REFF_ERR_OUT_OF_MEMORY} handle None out [0.0, 0.0, 0.0, 0.0] host memory" in r.stdout
