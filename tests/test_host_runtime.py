"""The library's host code against a HIP runtime without a device (host_hip.c): memory is the host's, kernels do nothing, and a
chosen call fails.  In a process of its own, which exits normally also where the host code would have used a null pointer."""
import os
import subprocess
import sys

import pytest

from paper_2502_09138_amd import tracker as trk

HERE = os.path.dirname(os.path.abspath(__file__))

MERGE = r"""
import ctypes as C, os, sys
import numpy as np
hip = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
hip.host_hip_of_size.restype, hip.host_hip_of_size.argtypes = C.c_void_p, [C.c_size_t]
from paper_2502_09138_amd import tracker as T
from paper_2502_09138_amd.config import default_config
L = T.load()
c, keep = T.make_config(default_config(), max_clusters=1000, max_sectors=2)
h = C.c_void_p()
assert L.tpc_tracker_create(C.byref(c), C.byref(h)) == 0, L.tpc_last_error()
R = len(keep[0])
off, y = np.zeros(2 * R + 1, np.uint32), np.zeros(4, np.float32)
off[1:] = 4
lo, hi = np.zeros(2, np.float32), np.ones(2, np.float32)
f = T._Frame()
f.n_sectors, f.n_rows, f.n_clusters, f.flags = 2, R, 4, T.TPC_IN_HOST
f.row_offsets, f.y, f.z, f.sector_z_lo, f.sector_z_hi = (a.ctypes.data for a in (off, y, y, lo, hi))
rid = C.c_uint64()
assert L.tpc_track_timeframe(h, C.byref(f), C.byref(rid)) == 0, L.tpc_last_error()
# the request's result header in pinned memory (48 bytes): one track, so that the outputs are exported
C.cast(hip.host_hip_of_size(48), C.POINTER(C.c_uint32))[2] = 1
before = hip.host_hip_mallocs(), hip.host_hip_device_pointers()
phys, m = (C.c_int32 * 2)(0, 1), T._Merged()
hip.host_hip_fail(sys.argv[2].encode(), int(sys.argv[3]))
first = L.tpc_merge_sectors(h, rid, phys, C.byref(m))
second = L.tpc_merge_sectors(h, rid, phys, C.byref(m))
third = L.tpc_merge_sectors(h, rid, phys, C.byref(m))
assert L.tpc_release(h, rid) == 0
print("status", first, second, third, "allocations", hip.host_hip_mallocs() - before[0], "device addresses",
      hip.host_hip_device_pointers() - before[1])
L.tpc_tracker_destroy(h)
print("left", hip.host_hip_mallocs() - hip.host_hip_frees())
"""


@pytest.fixture(scope="module")
def host_hip(tmp_path_factory):
    if not os.path.exists(trk.LIB_PATH):
        from paper_2502_09138_amd import build
        build.build()
    lib = str(tmp_path_factory.mktemp("host_hip") / "libhost_hip.so")
    subprocess.check_call(["gcc", "-shared", "-fPIC", "-O1", "-Wall", "-o", lib, os.path.join(HERE, "host_hip.c")])
    return lib


@pytest.mark.parametrize("name, nth", [("hipHostMalloc", 1), ("hipHostGetDevicePointer", 1), ("hipHostMalloc", 2), ("none", 0)])
def test_merge_after_a_failed_allocation(host_hip, name, nth):
    """A merge whose pinned buffers could not all be had fails, and the next one gets what is missing, once."""
    r = subprocess.run([sys.executable, "-c", MERGE, host_hip, name, str(nth)], capture_output=True, text=True, timeout=120,
                       cwd=os.path.dirname(HERE))
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)
    status = 0 if name == "none" else trk.TPC_E_NOMEM
    assert r.stdout.splitlines() == [f"status {status} 0 0 allocations 2 device addresses 1", "left 0"], r.stdout
