"""The device's default memory pool, which holds the library's scratch between
calls: a caller's own larger release threshold stays, and xct_cache_clear gives
the memory back.  Each case is a process of its own, as the pool is set up once."""

import os
import subprocess
import sys

import pytest

from tests.gpu_util import say

pytestmark = pytest.mark.gpu

CHILD = """
import ctypes, math, re, sys
import torch
import paper_2505_13955_amd as xct
import synth

own = int(sys.argv[1])
x = torch.ones((8, 128, 128), device="cuda")
xct.load_library()
path = re.search(r"/\\S*libamdhip64\\S*", open("/proc/self/maps").read()).group(0)
hip = ctypes.CDLL(path)
pool = ctypes.c_void_p()
assert hip.hipDeviceGetDefaultMemPool(ctypes.byref(pool), 0) == 0
THRESHOLD, RESERVED = 4, 5


def attribute(which):
    v = ctypes.c_uint64()
    assert hip.hipMemPoolGetAttribute(pool, which, ctypes.byref(v)) == 0
    return v.value


if own:
    assert hip.hipMemPoolSetAttribute(pool, THRESHOLD, ctypes.byref(ctypes.c_uint64(own))) == 0
g = synth.Geometry(n_angles=60, n_det=190, nx=128, ny=128, center=94.5)
p = xct.forward_project(x, g)
torch.cuda.synchronize()
print("threshold", attribute(THRESHOLD), "reserved", attribute(RESERVED), flush=True)
xct.xct_cache_clear()
print("cleared", attribute(RESERVED), flush=True)
"""


def _run(own):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", CHILD, str(own)], cwd=root, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr
    words = r.stdout.split()
    return {words[i]: int(words[i + 1]) for i in range(0, len(words), 2)}


def test_scratch_is_kept_and_given_back():
    say("default pool")
    got = _run(0)
    assert got["threshold"] == (1 << 30) + (1 << 28)
    assert got["reserved"] > 0 and got["cleared"] == 0


def test_a_larger_threshold_of_the_caller_stays():
    say("default pool with a threshold of the caller's")
    assert _run(1 << 34)["threshold"] == 1 << 34
