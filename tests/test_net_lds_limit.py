"""The CTR call refuses, before any launch, a net whose kernel needs more LDS than
the device gives a block.  The limit is asked of the HIP runtime; here
two functions of a small library loaded ahead of it answer in its place."""
import os
import subprocess
import sys

import pytest

from paper_1711_06505_amd import ams

SHIM = """
#include <stdlib.h>
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int attr, int dev) { (void)attr; (void)dev; *v = atoi(getenv("LDS_LIMIT")); return 0; }
"""

# the CTR call on 72-200-80-2: by the widths alone 77632 bytes, with the kernel's
# padded rows and scratch 79936
CALLS = """
import ctypes, sys
ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
class Net(ctypes.Structure):
    _fields_ = [("n_layers", ctypes.c_int32), ("dims", ctypes.c_int32 * 4)]
P = ctypes.c_void_p
def net(*d):
    return Net(len(d) - 1, (ctypes.c_int32 * 4)(*d))
ptrs = (P * 8)(*[0x1000] * 8)
f = lib.ams_ctr_fwd_bwd
f.argtypes = [P, ctypes.c_int32, ctypes.c_int32] + [P] * 13 + [ctypes.c_size_t, P]
n = net(72, 200, 80, 2)
w = (ctypes.c_int32 * 1)(72)
# (a workspace of no bytes: a net that is accepted stops there)
print(f(ctypes.byref(n), 16, 1, ptrs, w, 0x1000, ptrs, ptrs, None, 0x1000, 0x1000, ptrs, ptrs, None, None, 0x1000, 0,
        None))
"""
DIMS, WS = 4, 5


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    if not os.path.exists(ams.LIB_PATH):
        pytest.skip("libams.so not built")
    d = tmp_path_factory.mktemp("shim")
    src, so = d / "shim.c", d / "libshim.so"
    src.write_text(SHIM)
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(so), str(src)], check=True)
    return str(so)


@pytest.mark.parametrize("limit,status", [(77_631, DIMS), (77_632, DIMS), (79_935, DIMS), (79_936, WS), (163_840, WS)])
def test_ctr_need_is_checked(shim, limit, status):
    r = subprocess.run([sys.executable, "-c", CALLS, shim, ams.LIB_PATH], capture_output=True, text=True, timeout=120,
                       env={**os.environ, "LDS_LIMIT": str(limit)})
    assert r.returncode == 0, r.stderr
    assert int(r.stdout) == status
