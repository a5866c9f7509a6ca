"""The release threshold of the device's default memory pool, which per-call scratch comes from:
raised to 1 GiB, and left alone where the program has set more."""
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

CHILD = """
import ctypes, sys
import torch
from paper_2609_13846_amd import dtp
torch.cuda.init()
lib, pool = dtp.lib(), ctypes.c_void_p()
THRESHOLD = 4  # hipMemPoolAttrReleaseThreshold
for f, args in (("hipDeviceGetDefaultMemPool", [ctypes.POINTER(ctypes.c_void_p), ctypes.c_int]),
                ("hipMemPoolSetAttribute", [ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p]),
                ("hipMemPoolGetAttribute", [ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p])):
    getattr(lib, f).argtypes = args
def check(e):
    assert e == 0, e
check(lib.hipDeviceGetDefaultMemPool(ctypes.byref(pool), 0))
before = ctypes.c_uint64(int(sys.argv[1]))
check(lib.hipMemPoolSetAttribute(pool, THRESHOLD, ctypes.byref(before)))
A = torch.rand(64, device="cuda") + 0.1
dtp.dtp_encode_affinity_device(A, torch.empty(64, dtype=torch.int64, device="cuda"))
after = ctypes.c_uint64()
check(lib.hipMemPoolGetAttribute(pool, THRESHOLD, ctypes.byref(after)))
print("threshold", after.value)
"""


@pytest.mark.parametrize("before,after", [(0, 1 << 30), (1 << 40, 1 << 40)])
def test_pool_threshold_is_raised_and_never_lowered(before, after):
    print(f"[gpu] memory pool threshold {before}", flush=True)
    # a process of its own: the library looks at the threshold once
    run = subprocess.run([sys.executable, "-c", CHILD, str(before)], capture_output=True, text=True, timeout=110)
    assert run.returncode == 0, run.stderr[-3000:]
    assert f"threshold {after}" in run.stdout
