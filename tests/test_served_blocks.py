"""Blocks of the launch that holds both ADV field groups in a served round: one
per tile and group, none idle, in batches so large that a box is one segment long
(boxes of 16^3 are one tile then, of 32^3 four).  The library's host code on the
CPU over hip_stub.c."""
import subprocess
import sys

import pytest

from test_server_failures import ROOT, stub   # noqa: F401 (fixture)

CHILD = r"""
import ctypes, sys
stub = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
stub.stub_blocks.restype = ctypes.c_long
sys.path.insert(0, sys.argv[2])
import numpy as np
from paper_1608_08748_amd import binding as b
n, count = int(sys.argv[3]), int(sys.argv[4])
L = b.lib()
p = b.server_params(precision=b.FP64, max_slots=count, persistent=False)
room = count * b.server_box_bytes(p, (n, n, n)) + L.mhd_server_reserved_bytes()
raw = np.zeros(room + 256, dtype=np.uint8)
p.workspace, p.workspace_bytes = (raw.ctypes.data + 255) & ~255, room
h = ctypes.c_void_p()
assert L.mhd_server_create(ctypes.byref(p), ctypes.byref(h)) == b.MHD_OK
r = b.Request()
r.n[0] = r.n[1] = r.n[2] = n
r.steps, r.borrow = 2, 1
W = np.ones((10, n, n, n))
for _ in range(count):
    i = ctypes.c_uint64()
    assert L.mhd_server_submit(h, ctypes.byref(r), W.ctypes.data_as(ctypes.POINTER(ctypes.c_double)),
                               ctypes.byref(i)) == b.MHD_OK
assert L.mhd_server_progress(h, None, None) == b.MHD_OK
# three substages, two groups, tiles of 256 columns
print("blocks", stub.stub_blocks(b"k_manyINS_10BAdvXZPair"), 3 * 2 * count * (n * n // 256))
assert L.mhd_server_destroy(h) == b.MHD_OK
"""


@pytest.mark.parametrize("n, count", [(16, 256), (32, 64)])
def test_no_idle_blocks(stub, n, count):   # noqa: F811
    res = subprocess.run([sys.executable, "-c", CHILD, stub, ROOT, str(n), str(count)], capture_output=True,
                         text=True, timeout=120)
    assert res.returncode == 0, res.stdout + res.stderr
    got, tiles = res.stdout.split("blocks")[1].split()
    assert got == tiles, res.stdout
