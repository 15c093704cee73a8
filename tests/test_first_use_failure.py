"""A context whose first use fails on the device side (the table of the 1X1V
solver, the clearing of the slots) is left as it was: the same call made again
succeeds and no device memory is lost.  On the host: stubs of the HIP calls
that libvl.so makes, loaded ahead of it in a process of its own, count the
allocations and fail where told; no GPU is touched."""
import os
import subprocess
import sys

import pytest

from gpu_util import ensure_lib

STUB = r"""
#include <stdlib.h>
#include <string.h>
static int fail_at = -1, fallible = 0, live = 0;
void stub_fail_at(int k) { fail_at = k; fallible = 0; }
int stub_live(void) { return live; }
static int next_call(void) { return fallible++ == fail_at ? 999 : 0; }
int hipGetDeviceCount(int* n) { *n = 1; return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipMalloc(void** p, size_t n) { *p = malloc(n); ++live; return 0; }
int hipFree(void* p) { free(p); --live; return 0; }
int hipMemset(void* p, int v, size_t n) { int e = next_call(); if (!e) memset(p, v, n); return e; }
int hipLaunchKernel(const void* f, unsigned long long g0, unsigned g1, unsigned long long b0, unsigned b1, void** a,
                    size_t s, void* st) { return 0; }
int hipGetLastError(void) { return next_call(); }
int hipStreamSynchronize(void* s) { return next_call(); }
const char* hipGetErrorString(int e) { return "planted"; }
"""

CHILD = r"""
import ctypes, sys
sys.path.insert(0, sys.argv[3])
stub = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
import builtins
real = builtins.__import__
def no_torch(name, *a, **k):
    if name == "torch":
        raise ImportError(name)
    return real(name, *a, **k)
builtins.__import__ = no_torch
from paper_2109_06743_amd import vl, workloads as W
lib = vl.load()
at = int(sys.argv[2])
cfg, _ = W.landau(nx=16, nv=8)
c, h = vl.make_config(cfg, "f64"), ctypes.c_void_p()
assert lib.vl_create(ctypes.byref(c), ctypes.byref(h)) == 0
buf = ctypes.create_string_buffer(4096)
call = lambda: lib.vl_poisson(h, buf, ctypes.byref(buf, 2048), None)
stub.stub_fail_at(at)
first = call()
assert first == 5, (first, lib.vl_last_error(h))          # VL_EHIP
assert stub.stub_live() == 0, "device memory lost"
stub.stub_fail_at(-1)
again = call()
assert again == 0, (again, lib.vl_last_error(h))
lib.vl_destroy(h)
assert stub.stub_live() == 0
print("ok")
"""


@pytest.mark.parametrize("at", [0, 1, 2], ids=["memset", "launch", "synchronize"])
def test_first_use_can_be_repeated(at, tmp_path):
    ensure_lib()
    src, lib = tmp_path / "stub.c", tmp_path / "libstub.so"
    src.write_text(STUB)
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(lib), str(src)], check=True)
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", CHILD, str(lib), str(at), root], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr
