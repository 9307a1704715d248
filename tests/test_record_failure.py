"""lbm_record when a copy fails: the populations, the boundary state and the step count of the context
stay at one level, or the calls that would mix levels are refused.  No GPU: the library runs on a
stand-in for the HIP runtime, compiled here, whose device memory is host memory.  Its copies are real
and fail when told to; its only kernel is the step's, which adds 1 to the first boundary value of
side x0 on the way from one boundary region to the next, so that this value counts the levels.
"""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RUNTIME = r"""
#include <stddef.h>
#include <string.h>
typedef struct { unsigned x, y, z; } dim3_t;
int copies = 0, fail_from = 1 << 30, fail_to = 1 << 30;   /* copies [fail_from, fail_to) fail */
static struct { const void* f; int step; } known[4096];
static int nknown = 0;
static dim3_t cg, cb; static size_t csh; static void* cst;
static char scratch[1 << 21];
void** __hipRegisterFatBinary(const void* d) { static void* h; (void)d; return &h; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterFunction(void** m, const void* f, char* s, const char* name, unsigned n, void* a, void* b, void* c, void* d, int* e) {
    (void)m; (void)s; (void)n; (void)a; (void)b; (void)c; (void)d; (void)e;
    if (nknown < 4096) { known[nknown].f = f; known[nknown++].step = strstr(name, "k_step") != NULL; }
}
void __hipRegisterVar(void** m, void* v, char* h, char* d, int e, size_t s, int c, int g) { (void)m; (void)v; (void)h; (void)d; (void)e; (void)s; (void)c; (void)g; }
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t sh, void* st) { cg = g; cb = b; csh = sh; cst = st; return 0; }
int __hipPopCallConfiguration(dim3_t* g, dim3_t* b, size_t* sh, void** st) { *g = cg; *b = cb; *sh = csh; *st = cst; return 0; }
int hipLaunchKernel(const void* f, dim3_t g, dim3_t b, void** args, size_t sh, void* st) {
    (void)g; (void)b; (void)sh; (void)st;
    for (int k = 0; k < nknown; ++k)
        if (known[k].f == f && known[k].step) {   /* k_step(A, B, BndArgs, ..): reg_cur, reg_next behind 8 int, 3 of 8 bytes */
            double **reg = (double**)((char*)args[2] + 56);
            *reg[1] = *reg[0] + 1.0;
        }
    return 0;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void* st) {
    (void)kind; (void)st;
    const int k = copies++;
    if (k >= fail_from && k < fail_to) return 1;
    memmove(d, s, n);
    return 0;
}
int hipMemsetAsync(void* d, int v, size_t n, void* st) { (void)st; memset(d, v, n); return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetLastError(void) { return 0; }
const char* hipGetErrorString(int e) { (void)e; return "told to fail"; }
int hipGetSymbolAddress(void** p, const void* s) { (void)s; *p = scratch; return 0; }
int hipStreamSynchronize(void* s) { (void)s; return 0; }
int hipStreamIsCapturing(void* s, int* st) { (void)s; *st = 0; return 0; }
int hipStreamCreateWithFlags(void** s, unsigned f) { (void)f; *s = scratch; return 0; }
int hipStreamDestroy(void* s) { (void)s; return 0; }
int hipStreamWaitEvent(void* s, void* e, unsigned f) { (void)s; (void)e; (void)f; return 0; }
int hipEventCreate(void** e) { *e = scratch; return 0; }
int hipEventCreateWithFlags(void** e, unsigned f) { (void)f; *e = scratch; return 0; }
int hipEventDestroy(void* e) { (void)e; return 0; }
int hipEventRecord(void* e, void* s) { (void)e; (void)s; return 0; }
int hipEventSynchronize(void* e) { (void)e; return 0; }
int hipEventElapsedTime(float* t, void* a, void* b) { (void)a; (void)b; *t = 0; return 0; }
"""

PROGRAM = r"""
import ctypes, sys
import numpy as np
sys.path.insert(0, sys.argv[2])
rt = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)   # before the library: its symbols come first
from paper_2307_16766_amd import lbm
L = ctypes.CDLL(lbm.LIB_PATH)
vp, sz = ctypes.c_void_p, ctypes.c_size_t
for n in ("lbm_workspace_bytes", "lbm_tape_bytes", "lbm_state_bytes"):
    getattr(L, n).restype = sz
L.lbm_steps_done.restype = ctypes.c_long
L.lbm_last_error.restype = ctypes.c_char_p
L.lbm_init.argtypes = [vp, vp, sz, vp, vp, vp, vp, vp, vp]
L.lbm_record.argtypes = [vp, ctypes.c_int, ctypes.c_int, vp, sz]
L.lbm_step.argtypes = [vp, ctypes.c_int]
L.lbm_boundary_state.argtypes = [vp, ctypes.c_int, vp]
L.lbm_tape_bytes.argtypes = [vp, ctypes.c_int, ctypes.c_int]
for n in ("lbm_save", "lbm_restore"):
    getattr(L, n).argtypes = [vp, vp]
for n in ("lbm_steps_done", "lbm_state_bytes", "lbm_last_error", "lbm_destroy"):
    getattr(L, n).argtypes = [vp]
counter = {n: ctypes.c_int.in_dll(rt, n) for n in ("copies", "fail_from", "fail_to")}
OFF = 1 << 30

def aligned(n):
    a = np.zeros(n + 256, dtype=np.uint8)
    return a[(-a.ctypes.data) % 256:][:n]

NX, NY, N, EVERY = 20, 12, 7, 2
cfg = lbm.make_config(9, NX, NY, 0.7, ["lodi", "lodi", "periodic", "periodic"])
field = np.ones(NX * NY)

def context():
    n = L.lbm_workspace_bytes(ctypes.byref(cfg))
    ws, ctx = aligned(n), vp()
    p = field.ctypes.data
    assert L.lbm_init(ctypes.byref(cfg), ws.ctypes.data, n, None, p, p, p, p, ctypes.byref(ctx)) == 0
    return ws, ctx

def level(ctx):
    out = np.full(NY * 4, -1.0)
    rc = L.lbm_boundary_state(ctx, 0, out.ctypes.data)
    return rc, out[0]

def record(ctx, first, last):
    nt = L.lbm_tape_bytes(ctx, N, EVERY)
    tape = aligned(nt)
    counter["copies"].value, counter["fail_from"].value, counter["fail_to"].value = 0, first, last
    rc = L.lbm_record(ctx, N, EVERY, tape.ctypes.data, nt)
    ncopies = counter["copies"].value
    counter["fail_from"].value = counter["fail_to"].value = OFF
    return rc, ncopies

ws, ctx = context()
rc, total = record(ctx, OFF, OFF)
assert rc == 0 and level(ctx) == (0, N) and L.lbm_steps_done(ctx) == N
L.lbm_destroy(ctx)
stopped = set()
for k in range(total):
    for last in (k + 1, OFF):     # this copy alone fails, or every one from it on
        ws, ctx = context()
        saved = aligned(L.lbm_state_bytes(ctx))
        assert L.lbm_save(ctx, saved.ctypes.data) == 0
        rc, _ = record(ctx, k, last)
        assert rc == lbm.LBM_E_HIP, (k, rc)
        assert b"told to fail" in L.lbm_last_error(ctx)
        n = L.lbm_steps_done(ctx)
        stopped.add(n)
        rc, at = level(ctx)
        if rc == 0:
            assert at == n, (k, last, at, n)
            assert L.lbm_step(ctx, 2) == 0 and level(ctx) == (0, n + 2)
        else:                     # the copy back failed too (or it was the one told to)
            assert rc == lbm.LBM_E_STATE and (last == OFF or k == total - 1), (k, last, rc)
            assert L.lbm_step(ctx, 1) == lbm.LBM_E_STATE and L.lbm_save(ctx, saved.ctypes.data) == lbm.LBM_E_STATE
            assert L.lbm_steps_done(ctx) == n
        assert L.lbm_restore(ctx, saved.ctypes.data) == 0 and level(ctx) == (0, 0)
        assert L.lbm_step(ctx, 1) == 0 and level(ctx) == (0, 1)
        L.lbm_destroy(ctx)
assert stopped == {0, 2, 4, 6, N}, stopped
print("checked", total)
"""


def test_failed_copies_leave_one_level(tmp_path):
    src, lib = tmp_path / "runtime.c", tmp_path / "runtime.so"
    src.write_text(RUNTIME)
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", str(src), "-o", str(lib)], check=True)
    r = subprocess.run([sys.executable, "-c", PROGRAM, str(lib), ROOT], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.startswith("checked 1")
