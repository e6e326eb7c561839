"""A stand-in for the HIP runtime, built from C, and a process that runs the
library on it: for tests of host code without a device.

Allocations are numbers out of a limited address range.  Kernels are not run;
their launches and arguments are recorded.  Copies out of pinned memory are
queued and read as late as the library's waits allow; one whose source has
changed by then is counted."""

import json
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STAND_IN = r"""
#include <stddef.h>
#include <stdint.h>
#include <string.h>
typedef struct { unsigned x, y, z; } dim3_;
typedef void (*hook_t)(const char *, unsigned, unsigned, unsigned, unsigned, void **);
enum { MAXP = 4096 };
static struct { uintptr_t p; size_t n; } blk[MAXP];
static int nblk;
static size_t used, limit = ~(size_t)0;
static uintptr_t next = 0x100000000000ull;
static hook_t hook;
static struct { const void *f; const char *name; } fn[MAXP];
static int nfn;
static char pinned[8 << 20];
static size_t pinned_used;
static int capturing;
void stand_in(size_t lim, hook_t h) { limit = lim; hook = h; }
size_t stand_in_used(void) { return used; }
size_t stand_in_block(uintptr_t p) { for (int i = 0; i < nblk; i++) if (blk[i].p <= p && p < blk[i].p + blk[i].n) return blk[i].p + blk[i].n - p; return 0; }
int hipMalloc(void **p, size_t n) {
    if (used + n > limit || nblk == MAXP) { *p = 0; return 2; }
    *p = (void *)next; blk[nblk].p = next; blk[nblk].n = n; nblk++; next += (n + 0xfffff) & ~(size_t)0xfffff; used += n;
    return 0;
}
int hipFree(void *p) {
    for (int i = 0; i < nblk; i++) if (blk[i].p == (uintptr_t)p) { used -= blk[i].n; blk[i] = blk[--nblk]; return 0; }
    return 1;
}
int hipHostMalloc(void **p, size_t n, unsigned f) { if (pinned_used + n > sizeof pinned) return 2; *p = pinned + pinned_used; pinned_used += n; return 0; }
int hipHostFree(void *p) { return 0; }
/* the stream's pending copies out of pinned memory, with their sources' sums when queued */
static struct { const unsigned char *s; size_t n; uint64_t sum; } cp[1 << 16];
static int ncp, done, bad, nev, ev_pos[MAXP];
static uint64_t sum_of(const unsigned char *s, size_t n) { uint64_t h = 1469598103934665603ull; for (size_t i = 0; i < n; i++) h = (h ^ s[i]) * 1099511628211ull; return h; }
static void retire(int to) { for (; done < to; done++) bad += sum_of(cp[done].s, cp[done].n) != cp[done].sum; }
int stand_in_copies(void) { return ncp; }
int stand_in_pending(void) { return ncp - done; }
int stand_in_bad(void) { return bad; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *st) {
    if (kind == 2) memset(d, 0, n);
    else if ((const char *)s >= pinned && (const char *)s < pinned + sizeof pinned && ncp < 1 << 16) { cp[ncp].s = s; cp[ncp].n = n; cp[ncp].sum = sum_of(s, n); ncp++; }
    return 0;
}
int hipMemcpy(void *d, const void *s, size_t n, int kind) { if (kind == 2) memset(d, 0, n); return 0; }
int hipMemset(void *p, int v, size_t n) { return 0; }
int hipMemsetAsync(void *p, int v, size_t n, void *s) { return 0; }
int hipGetDeviceCount(int *n) { *n = 1; return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipSetDevice(int d) { return 0; }
int hipGetDevicePropertiesR0600(void *p, int d) { memset(p, 0, 64); return 0; }
int hipGetLastError(void) { return 0; }
const char *hipGetErrorString(int e) { return "stand-in"; }
int hipGetSymbolAddress(void **p, const void *s) { *p = (void *)0x200000000000ull; return 0; }
int hipFuncSetAttribute(const void *f, int a, int v) { return 0; }
int hipEventCreate(void **e) { if (nev + 1 >= MAXP) return 2; *e = (void *)(uintptr_t)++nev; return 0; }
int hipEventCreateWithFlags(void **e, unsigned f) { return hipEventCreate(e); }
int hipEventDestroy(void *e) { return 0; }
int hipEventRecord(void *e, void *s) { ev_pos[(uintptr_t)e] = ncp; return 0; }
int hipEventSynchronize(void *e) { retire(ev_pos[(uintptr_t)e]); return 0; }
int hipEventElapsedTime(float *t, void *a, void *b) { *t = 0; return 0; }
int hipStreamCreateWithFlags(void **s, unsigned f) { *s = (void *)2; return 0; }
int hipStreamDestroy(void *s) { return 0; }
int hipStreamSynchronize(void *s) { retire(ncp); return 0; }
int hipStreamIsCapturing(void *s, int *c) { *c = capturing; return 0; }
int hipStreamBeginCapture(void *s, int m) { capturing = 1; return 0; }
int hipStreamEndCapture(void *s, void **g) { capturing = 0; *g = (void *)3; return 0; }
int hipGraphGetNodes(void *g, void **n, size_t *c) { *c = 1; return 0; }
int hipGraphInstantiate(void **e, void *g, void *a, char *b, size_t n) { *e = (void *)4; return 0; }
int hipGraphLaunch(void *e, void *s) { if (hook) hook("graph", 0, 0, 0, 0, 0); return 0; }
int hipGraphDestroy(void *g) { return 0; }
int hipGraphExecDestroy(void *e) { return 0; }
static struct { dim3_ g, b; size_t shm; void *s; } cfg;
int __hipPushCallConfiguration(dim3_ g, dim3_ b, size_t shm, void *s) { cfg.g = g; cfg.b = b; cfg.shm = shm; cfg.s = s; return 0; }
int __hipPopCallConfiguration(dim3_ *g, dim3_ *b, size_t *shm, void **s) { *g = cfg.g; *b = cfg.b; *shm = cfg.shm; *s = cfg.s; return 0; }
void **__hipRegisterFatBinary(const void *d) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **m) {}
void __hipRegisterFunction(void **m, const void *f, char *dev, const char *name, unsigned n, void *a, void *b, void *c, void *d, int *w) { if (nfn < MAXP) { fn[nfn].f = f; fn[nfn].name = name; nfn++; } }
void __hipRegisterVar(void **m, void *v, char *h, char *d, int e, size_t n, int c, int g) {}
int hipLaunchKernel(const void *f, dim3_ g, dim3_ b, void **args, size_t shm, void *s) {
    const char *name = "?";
    for (int i = 0; i < nfn; i++) if (fn[i].f == f) name = fn[i].name;
    if (hook) hook(name, g.x, g.y, g.z, b.x, args);
    return 0;
}
"""

# runs in a process of its own, without torch: argv[1] the C stand-in, argv[2] the library, argv[3] the scenario
DRIVER = r"""
import ctypes, json, sys
import numpy as np
hip, rp = ctypes.CDLL(sys.argv[1]), ctypes.CDLL(sys.argv[2])
P, I, D, Z, L = ctypes.c_void_p, ctypes.c_int, ctypes.c_double, ctypes.c_size_t, ctypes.c_long
hip.stand_in_used.restype = hip.stand_in_block.restype = Z
hip.stand_in_block.argtypes = [P]
class Cell(ctypes.Structure):
    _fields_ = [("lat", D * 9), ("fft", I * 3), ("kmesh", I * 3)]
class Problem(ctypes.Structure):
    _fields_ = [("cell", Cell), ("iq", I * 3), ("nband", I), ("npw_max", I), ("npw", P), ("mmax", I * 3), ("miller", P),
                ("coef", P), ("energy", P), ("T", P), ("o0", I), ("o1", I), ("e0", I), ("e1", I), ("k0", I), ("k1", I),
                ("ng", I), ("gsph", P), ("nfreq", I), ("freq", P), ("delta", D), ("wm", I), ("kbatch", I),
                ("accumulate", I), ("chi", P)]
def cell(n, k): return Cell((D * 9)(7, 0, 0, 0, 7, 0, 0, 0, 7), (I * 3)(n, n, n), (I * 3)(*k))
def sphere(n):
    r = np.arange(-8, 9)
    m = np.stack(np.meshgrid(r, r, r, indexing="ij"), -1).reshape(-1, 3)
    return np.ascontiguousarray(m[np.argsort((m ** 2).sum(1), kind="stable")][1:n + 1].astype(np.int32))
def ptr(a): return a.ctypes.data_as(P)
launches = []
HOOK = ctypes.CFUNCTYPE(None, ctypes.c_char_p, *[ctypes.c_uint] * 4, ctypes.POINTER(P))
def arg(args, i, t): return ctypes.cast(args[i], ctypes.POINTER(t))[0]
def record(name, x, y, z, b, args):
    n, rec = name.decode(), None
    if "k_chi_f64_sum" in n: rec = dict(k="sum", nfreq=arg(args, 1, I), nslice=arg(args, 2, I))
    elif "k_chi_f64" in n:
        ng, nf, ns, out = arg(args, 1, I), arg(args, 3, I), arg(args, 7, I), arg(args, 8, P)
        rec = dict(k="chi", nfreq=nf, nslice=ns, y=y, need=16 * ns * nf * ng * ng, room=hip.stand_in_block(out))
    elif "k_ugrid_planes" in n: rec = dict(k="ugrid", bands=y, n=z, room=hip.stand_in_block(arg(args, 13, P)))
    elif "k_gj_first" in n: rec = dict(k="gj", nmat=y, room=hip.stand_in_block(arg(args, 3, P)))
    elif n == "graph": rec = dict(k="graph")
    if rec: launches.append(rec)
hook = HOOK(record)
ctx, big, one = P(), P(0x300000000000), np.ones(1)
assert rp.rp_create(ctypes.byref(ctx), 0, None) == 0
def limit(extra): hip.stand_in(Z(hip.stand_in_used() + extra), hook)
def accumulate(npair, ng, nfreq):
    f = np.linspace(0.0, 9.0, nfreq) + 0j
    return rp.rp_chi0_accumulate(ctx, ctypes.byref(cell(16, (1, 1, 1))), (I * 3)(0, 0, 0), 1 + npair, big, None, 0, 1, 1,
                                 1 + npair, 0, 1, ng, big, nfreq, ptr(f), D(0.1), 1, 0, 0, big)
def bands(nk, npw): return np.full(nk, npw, np.int32)
def pair(kmesh, n, nocc, nemp, ng, prec):
    nk, g = int(np.prod(kmesh)), sphere(ng)
    return rp.rp_pair_density(ctx, ctypes.byref(cell(n, kmesh)), (I * 3)(0, 0, 0), nocc + nemp, 60, ptr(bands(nk, 60)),
                              (I * 3)(8, 8, 8), big, big, 0, nocc, nocc, nocc + nemp, 0, nk, ng, ptr(g), prec, big)
def problem(kmesh, n, nocc, nemp, ng, nfreq, kbatch, keep):
    nk, g, w, f = int(np.prod(kmesh)), sphere(ng), bands(int(np.prod(kmesh)), 60), np.linspace(0.0, 9.0, nfreq) + 0j
    keep += [g, w, f]
    return Problem(cell(n, kmesh), (I * 3)(0, 0, 0), nocc + nemp, 60, ptr(w), (I * 3)(8, 8, 8), big, big, big, None, 0, nocc,
                   nocc, nocc + nemp, 0, nk, ng, ptr(g), nfreq, ptr(f), 0.1, 1, kbatch, 0, big)
def screen(ng, nfreq):
    return rp.rp_screen_W(ctx, ctypes.byref(cell(16, (1, 1, 1))), (I * 3)(0, 0, 0), ng, ptr(sphere(ng)), nfreq, big, big, None)
MB = 1 << 20
out = []
def call(extra, fn, *a):
    launches.clear()
    limit(extra)
    st = fn(*a)
    rp.rp_last_error.restype = ctypes.c_char_p
    out.append(dict(status=st, err=rp.rp_last_error(ctx).decode(), launches=list(launches)))
exec(sys.argv[3])
print(json.dumps(out))
"""


def build(d):
    """A function that runs a scenario (Python text after DRIVER's) in a process
    of its own and returns what it recorded; files go to folder d."""
    cc = shutil.which("gcc") or shutil.which("cc")
    lib = os.path.join(ROOT, "paper_2001_02351_amd", "librp.so")
    if cc is None:
        pytest.skip("no host C compiler")
    if not os.path.exists(lib):
        from paper_2001_02351_amd.build import build
        build()
    (d / "hip.c").write_text(STAND_IN)
    so = d / "libamdhip64.so.7"
    subprocess.run([cc, "-shared", "-fPIC", "-O1", "-w", str(d / "hip.c"), "-o", str(so)], check=True)
    (d / "driver.py").write_text(DRIVER)

    def run(scenario):
        env = dict(os.environ, LD_LIBRARY_PATH=str(d))
        p = subprocess.run([sys.executable, str(d / "driver.py"), str(so), lib, scenario], env=env, capture_output=True,
                           text=True, timeout=120)
        assert p.returncode == 0, p.stderr
        return json.loads(p.stdout)

    return run
