"""Kernels that take more than 64 KB of dynamic LDS: the limit is raised on every device that
launches them, and an error of raising it is returned.  The HIP calls go to a stand-in that
records them (the machine that runs this needs no GPU); each test has a process of its own."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2403_06082_amd", "libfq.so")

STAND_IN = r"""
#include <stddef.h>
#include <string.h>
typedef struct { unsigned x, y, z; } dim3;
static int dev, fail, launches, large, bad, nset;
static dim3 G, B; static size_t S; static void* T;
static struct { const void* f; int dev, bytes; } set[256];
void stand_in(int device, int error) { dev = device; fail = error; launches = large = bad = 0; }
void counts(int* out) { out[0] = launches; out[1] = large; out[2] = bad; }
int hipGetDevice(int* d) { *d = dev; return 0; }
int hipDeviceGetAttribute(int* v, int a, int d) { *v = 256; return 0; }
int hipGetLastError(void) { return 0; }
const char* hipGetErrorString(int e) { return "stand-in"; }
int hipFuncSetAttribute(const void* f, int a, int v) {
  if (fail) return fail;
  if (nset < 256) { set[nset].f = f; set[nset].dev = dev; set[nset++].bytes = v; }
  return 0;
}
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, void* t) { G = g; B = b; S = s; T = t; return 0; }
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, void** t) { *g = G; *b = B; *s = S; *t = T; return 0; }
int hipLaunchKernel(const void* f, dim3 g, dim3 b, void** a, size_t lds, void* t) {
  ++launches;
  if (lds > 65536) {
    int ok = 0;
    ++large;
    for (int i = 0; i < nset; ++i) ok |= set[i].f == f && set[i].dev == dev && (size_t)set[i].bytes >= lds;
    bad += !ok;
  }
  return 0;
}
"""

CHILD = r"""
import ctypes, sys
H = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
L = ctypes.CDLL(sys.argv[2])
i64, P = ctypes.c_int64, ctypes.c_void_p
class TFF(ctypes.Structure):
    _fields_ = [("d", i64), ("k", i64), ("rho", i64), ("R1", P), ("d1", i64), ("R2", P), ("d2", i64)]
for n in ("fq_tff_analysis", "fq_tff_synthesis", "fq_frame_analysis_tff"):
    getattr(L, n + "_workspace_bytes").restype = ctypes.c_size_t
A = P(1 << 20)                       # never read: no kernel runs
wide = TFF(13824, 950, 16, A, 108, A, 128)
few = TFF(4000, 2000, 2, A, 50, A, 80)        # four vectors of 2000 subspaces a work-group
def calls(f):
    ref = ctypes.byref(f)
    out = []
    for n in (1, 3, 17):
        out.append(L.fq_tff_synthesis(None, A, i64(n), ref, A, A, ctypes.c_size_t(1 << 40)))
        out.append(L.fq_tff_analysis(None, A, 0, i64(n), i64(f.d), ref, A, A, ctypes.c_size_t(1 << 40)))
    out.append(L.fq_frame_analysis_tff(None, A, 0, ref, ref, A, A, A, A, ctypes.c_size_t(1 << 40)))
    return out
for f in (wide, few):
    for device in (0, 1, 0):
        H.stand_in(device, 0)
        assert calls(f) == [0] * 7
        c = (ctypes.c_int * 3)()
        H.counts(c)
        assert c[1] > 0 and c[2] == 0, (device, f.d, list(c))
    H.stand_in(2, 98)                # raising the limit fails: the call says so
    assert 6 in calls(f)
    c = (ctypes.c_int * 3)()
    H.counts(c)
    assert c[1] == 0, list(c)        # and nothing was launched beyond the limit
print("ok")
"""


@pytest.mark.skipif(not shutil.which("gcc"), reason="needs a C compiler")
def test_limit_on_every_device_and_its_error(tmp_path):
    src, so = tmp_path / "hip.c", tmp_path / "libhip_stand_in.so"
    src.write_text(STAND_IN)
    subprocess.run(["gcc", "-shared", "-fPIC", "-w", "-o", str(so), str(src)], check=True)
    r = subprocess.run([sys.executable, "-c", CHILD, str(so), LIB], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "ok" in r.stdout, r.stdout + r.stderr
