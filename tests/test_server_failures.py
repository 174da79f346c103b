"""Served rounds whose report fails for want of host memory: the library's host
code on the CPU over hip_stub.c, in a process of its own.  Every request is
reported once, with its own totals slot, whatever failed before, and the server
can be destroyed at any point."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

CHILD = r"""
import ctypes, sys
stub = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
import numpy as np
from paper_1608_08748_amd import binding as b
L = b.lib()
p = b.server_params(precision=b.FP64, max_slots=8)
size = 64 << 20
raw = np.zeros(size + L.mhd_server_reserved_bytes() + 256, dtype=np.uint8)
p.workspace = (raw.ctypes.data + 255) & ~255
p.workspace_bytes = size + L.mhd_server_reserved_bytes()
h = ctypes.c_void_p()
assert L.mhd_server_create(ctypes.byref(p), ctypes.byref(h)) == b.MHD_OK
D = ctypes.POINTER(ctypes.c_double)

def submit(n, steps):
    r = b.Request()
    r.n[0], r.n[1], r.n[2], r.steps, r.keep_state = 4, 4, n, steps, 1
    W = np.ones((10, n, 4, 4))
    i = ctypes.c_uint64()
    assert L.mhd_server_submit(h, ctypes.byref(r), W.ctypes.data_as(D), ctypes.byref(i)) == b.MHD_OK
    return i.value, n

def progress():
    a, q = ctypes.c_int(), ctypes.c_int()
    return L.mhd_server_progress(h, ctypes.byref(a), ctypes.byref(q))

def poll():
    buf, n = (b.Completion * 16)(), ctypes.c_int()
    assert L.mhd_server_poll(h, buf, 16, ctypes.byref(n)) == b.MHD_OK
    assert all(buf[k].status == b.MHD_OK for k in range(n.value))
    return [(buf[k].id, buf[k].steps, buf[k].cells) for k in range(n.value)]

want = [submit(n, s) + (s,) for n, s in ((4, 1), (8, 1), (5, 1), (6, 2), (7, 3))]
def set_stub(name, kind, v): kind.in_dll(stub, name).value = v
# the report of the second box finds no memory for its state, then once more
set_stub("stub_new_bytes", ctypes.c_size_t, 11 * 8 * 16 * 8)
assert progress() == b.MHD_OK and poll() == []
got = []
for fails in range(2):
    set_stub("stub_fail_new", ctypes.c_int, 1)
    assert progress() == b.MHD_ENOMEM, "the allocation was not asked for"
    got += poll()
    assert [g[0] for g in got] == [want[0][0]], got
if sys.argv[3] == "go on":
    for _ in range(6):
        assert progress() == b.MHD_OK
        got += poll()
    assert got == [(i, s, 16 * n) for i, n, s in want], (got, want)
    used = ctypes.c_size_t(1)
    assert L.mhd_server_memory(h, ctypes.byref(used), None, None) == b.MHD_OK and used.value == 0
    for i, n, s in want:
        out = np.empty((11, n, 4, 4))
        assert L.mhd_server_result(h, i, out.ctypes.data_as(D), out.size) == b.MHD_OK
assert L.mhd_server_destroy(h) == b.MHD_OK
print("done")
"""


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("stub") / "hip_stub.so")
    subprocess.check_call(["gcc", "-O1", "-fPIC", "-shared", "-w", os.path.join(HERE, "hip_stub.c"), "-o", so])
    return so


@pytest.mark.parametrize("then", ["go on", "destroy"])
def test_report_without_memory(stub, then):
    res = subprocess.run([sys.executable, "-c", CHILD, stub, ROOT, then], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0 and "done" in res.stdout, res.stdout + res.stderr
