"""mhd_get_state where its pinned slots cannot serve: the library's host code on
the CPU over hip_stub.c.  On a stream of another device than the slots' events
the runtime copies; under capture the call is refused and leaves the caller's
memory alone, the first time and once the slots are there."""
import os
import subprocess
import sys

from test_server_failures import ROOT, stub   # noqa: F401 (fixture)

CHILD = r"""
import ctypes, sys
stub = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
import numpy as np
from paper_1608_08748_amd import binding as b
L = b.lib()
D = ctypes.POINTER(ctypes.c_double)

def set_stub(name, v):
    ctypes.c_int.in_dll(stub, name).value = v

shape = (40, 50, 60)
for case in ("other device", "capture first", "capture later"):
    p = b.make_params(shape, precision=b.FP64)
    size = L.mhd_workspace_bytes(ctypes.byref(p))
    raw = np.zeros(size + 256, dtype=np.uint8)
    p.workspace, p.workspace_bytes = (raw.ctypes.data + 255) & ~255, size
    h = ctypes.c_void_p()
    assert L.mhd_create(ctypes.byref(p), ctypes.byref(h)) == b.MHD_OK
    out = np.full((11,) + shape, 7.0)
    get = lambda: L.mhd_get_state(h, out.ctypes.data_as(D))
    if case == "other device":
        set_stub("stub_other_device", 1)
        assert get() == b.MHD_OK and (out == 0).all()
        set_stub("stub_other_device", 0)
    else:
        if case == "capture later":
            assert get() == b.MHD_OK and (out == 0).all()
            out[:] = 7.0
        set_stub("stub_capturing", 1)
        assert get() == b.MHD_EDEVICE and (out == 7).all(), case
        set_stub("stub_capturing", 0)
        assert get() == b.MHD_OK and (out == 0).all()
    assert L.mhd_destroy(h) == b.MHD_OK
print("done")
"""


def test_where_the_slots_cannot_serve(stub):   # noqa: F811
    res = subprocess.run([sys.executable, "-c", CHILD, stub, ROOT], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0 and "done" in res.stdout, res.stdout + res.stderr
