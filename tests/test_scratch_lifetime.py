"""Scratch of whmc_apply_MdagM over calls of growing and shrinking numbers of right-hand sides: a captured graph
holds the addresses of the buffers of its calls, so none may be freed before the context is destroyed.  CPU
only: the library's host code runs on a stand-in for the HIP runtime that hands out addresses, counts what is
freed and launches nothing."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1805_03560_amd", "libwhmc.so")

STUB = r"""
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
typedef struct { unsigned x, y, z; } dim3_;
static size_t next = 0x100000, used, limit = (size_t)-1, allocs, frees;
static int capturing;
size_t stub_used(void) { return used; }
size_t stub_allocs(void) { return allocs; }
size_t stub_frees(void) { return frees; }
void stub_limit(size_t b) { limit = b; }
void stub_capture(int on) { capturing = on; }
int hipMalloc(void** p, size_t n) {
  if (capturing || n > limit) return 2;
  *p = (void*)next;
  next += (n + 4095) / 4096 * 4096 + 4096;
  used += n, ++allocs;
  return 0;
}
int hipFree(void* p) { if (p) ++frees; return 0; }
int hipHostMalloc(void** p, size_t n, unsigned f) { (void)f; *p = calloc(1, n); return 0; }
int hipHostFree(void* p) { free(p); return 0; }
int hipStreamIsCapturing(void* s, int* st) { (void)s; *st = capturing; return 0; }
int hipSetDevice(int d) { (void)d; return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetDeviceCount(int* n) { *n = 1; return 0; }
int hipGetLastError(void) { return 0; }
int hipPeekAtLastError(void) { return 0; }
const char* hipGetErrorString(int e) { (void)e; return "stub"; }
int hipStreamSynchronize(void* s) { (void)s; return 0; }
int hipDeviceGetAttribute(int* v, int a, int d) { (void)a; (void)d; *v = 65536; return 0; }
int hipMemsetAsync(void* p, int v, size_t n, void* s) { (void)p; (void)v; (void)n; (void)s; return 0; }
int hipMemcpyAsync(void* d, const void* a, size_t n, int k, void* s) { (void)d; (void)a; (void)n; (void)k; (void)s; return 0; }
int hipGetSymbolAddress(void** p, const void* s) { (void)s; *p = (void*)0x1000; return 0; }
int __hipPushCallConfiguration(dim3_ g, dim3_ b, size_t m, void* s) { (void)g; (void)b; (void)m; (void)s; return 0; }
int __hipPopCallConfiguration(dim3_* g, dim3_* b, size_t* m, void** s) {
  memset(g, 0, sizeof *g); memset(b, 0, sizeof *b); *m = 0; *s = 0;
  return 0;
}
int hipLaunchKernel(const void* f, dim3_ g, dim3_ b, void** a, size_t m, void* s) {
  (void)f; (void)g; (void)b; (void)a; (void)m; (void)s;
  return 0;
}
void** __hipRegisterFatBinary(const void* d) { static void* h[4]; (void)d; return h; }
void __hipUnregisterFatBinary(void** h) { (void)h; }
void __hipRegisterFunction(void** h, const void* f, char* d, const char* n, unsigned t, void* a, void* b, void* c, void* e, int* w) {
  (void)h; (void)f; (void)d; (void)n; (void)t; (void)a; (void)b; (void)c; (void)e; (void)w;
}
void __hipRegisterVar(void** h, void* v, char* n, char* d, int e, size_t s, int c, int g) {
  (void)h; (void)v; (void)n; (void)d; (void)e; (void)s; (void)c; (void)g;
}
"""

DRIVER = r"""
import ctypes, sys
stub = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)   # before the library, so that its calls find these
L = ctypes.CDLL(sys.argv[2])
dims, counts = [int(v) for v in sys.argv[3].split(",")], [int(v) for v in sys.argv[4].split(",")]
for f in ("stub_used", "stub_allocs", "stub_frees"):
    getattr(stub, f).restype = ctypes.c_size_t
stub.stub_limit.argtypes = [ctypes.c_size_t]
P, D = ctypes.c_void_p, ctypes.c_double
ctx = P()
def ok(rc): assert rc == 0, rc
ok(L.whmc_create(ctypes.byref(ctx), (ctypes.c_int * 4)(*dims), 0, P(16)))
ok(L.whmc_load_gauge(ctx, P(0x2000), D(0.0)))
def call(n, eo): return L.whmc_apply_MdagM(ctx, P(0x3000), P(0x4000), (D * n)(*[0.1] * n), n, eo)
per = dims[0] * dims[1] * dims[2] * dims[3] * 192
for eo in (1, 0):
    used, frees = stub.stub_used(), stub.stub_frees()
    for n in counts:
        ok(call(n, eo))
        assert stub.stub_frees() == frees, "a buffer of an earlier call was freed"
    held = stub.stub_used() - used
    assert held <= 31 * per
    # captured calls and calls without memory make do with what there is
    allocs = stub.stub_allocs()
    stub.stub_capture(1)
    for n in counts + [16]: ok(call(n, eo))
    stub.stub_capture(0)
    stub.stub_limit(0)
    for n in counts + [16]: ok(call(n, eo))
    stub.stub_limit(ctypes.c_size_t(-1).value)
    assert stub.stub_allocs() == allocs and stub.stub_frees() == frees
L.whmc_destroy(ctx)
assert stub.stub_frees() == stub.stub_allocs()
print("ok")
"""


def _run(tmp_path, driver, dims, counts):
    src = tmp_path / "stub.c"
    src.write_text(STUB)
    stub = str(tmp_path / "stub.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-w", str(src), "-o", stub], check=True)
    r = subprocess.run([sys.executable, "-c", driver, stub, LIB, ",".join(map(str, dims)), ",".join(map(str, counts))],
                       capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stderr[-2000:]


DRIVER_BATCH = DRIVER[:DRIVER.index("for eo in")] + r"""
L.whmc_set_option.argtypes = [P, ctypes.c_int, ctypes.c_longlong]
ok(L.whmc_set_option(ctx, 2, 0))    # WHMC_OPT_HOP_SCHEDULE
used = stub.stub_used()
ok(call(4, 1))
assert stub.stub_used() - used == 4 * per
print("ok")
"""


# the direction-split kernels (eo = 1 and 0), the sweep kernels and the largest lattices' batches of four
@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (16, 16, 16, 16), (48, 24, 24, 24)])
@pytest.mark.parametrize("counts", [(1, 3, 16, 2), (3, 9), (1, 2, 4, 8, 16, 1), (20, 1)])
def test_no_scratch_of_an_earlier_call_is_freed(tmp_path, dims, counts):
    _run(tmp_path, DRIVER, dims, counts)


def test_several_masses_share_a_pass_whatever_the_schedule(tmp_path):
    """large lattices: an explicit schedule of the single-RHS kernels does not take the batches away"""
    _run(tmp_path, DRIVER_BATCH, (48, 24, 24, 24), (4,))
