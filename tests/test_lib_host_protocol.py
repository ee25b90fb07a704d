"""The host side of the library against a HIP runtime of this test's own (a
shared object that notes the kernels launched and fails copies on demand, loaded
before libmbkk.so in a process of its own): what a call that failed half-way
leaves behind.  No device is needed."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RUNTIME = r"""
#define _GNU_SOURCE
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
typedef struct { uint32_t x, y, z; } dim3;
static struct { const void *fn; const char *name; } reg[4096];
static int nreg, fail_d2d, nlog;
static const char *log_[4096];
static void *mods[64];
static int nmod;
void **__hipRegisterFatBinary(const void *d) { (void)d; return &mods[nmod++ & 63]; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterFunction(void **m, const void *fn, char *a, const char *name, unsigned b, void *c, void *d, void *e,
                           void *f, int *g)
{
    if (nreg < 4096) { reg[nreg].fn = fn; reg[nreg++].name = name; }
}
void __hipRegisterVar(void **m, void *v, char *a, char *b, int c, size_t d, int e, int f) {}
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, void *st) { return 0; }
int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *s, void **st)
{
    dim3 one = {1, 1, 1};
    *g = *b = one; *s = 0; *st = 0;
    return 0;
}
int hipLaunchKernel(const void *fn, dim3 g, dim3 b, void **args, size_t s, void *st)
{
    for (int i = 0; i < nreg; ++i)
        if (reg[i].fn == fn && nlog < 4096)
            log_[nlog++] = reg[i].name;
    return 0;
}
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *st)
{
    if (kind == 3 && fail_d2d)
        return 1;
    memcpy(d, s, n);
    return 0;
}
int hipGetLastError(void) { return 0; }
const char *hipGetErrorString(int e) { return e ? "as asked" : "none"; }
int hipStreamSynchronize(void *st) { return 0; }
int hipThreadExchangeStreamCaptureMode(int *m) { return 0; }
int hipHostMalloc(void **p, size_t n, unsigned f) { *p = calloc(1, n); return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
void fake_fail_d2d(int on) { fail_d2d = on; }
int fake_launched(const char *part)
{
    int n = 0;
    for (int i = 0; i < nlog; ++i)
        n += strstr(log_[i], part) != 0;
    nlog = 0;
    return n;
}
"""

PRELUDE = r"""
import ctypes as C, sys
sys.path.insert(0, sys.argv[2])
F = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
from paper_2410_05902_amd import _lib as L
lib = L.lib()
def ctx(**kw):
    base = dict(n=256, d=32, k=4, b_max=64, window=2, kernel=L.GAUSS, kernel_param=1.0, precision=L.FP32,
                lr=L.LR_BETA, cross_impl=L.CROSS_AUTO, tie_delta=0.0, validate=1)
    base.update(kw)
    cfg, nb, c = L.Config(**base), C.c_size_t(), C.c_void_p()
    L.check(lib.mbkk_workspace_size(C.byref(cfg), C.byref(nb)))
    ws = C.create_string_buffer(nb.value + 256)
    p = (C.addressof(ws) + 255) // 256 * 256
    L.check(lib.mbkk_create(C.byref(cfg), C.c_void_p(p), nb, None, C.byref(c)))
    X = (C.c_float * (cfg.n * cfg.d))()
    L.check(lib.mbkk_set_data(c, X, cfg.d), c)
    return c, (ws, X)
"""


def _run(tmp_path, body):
    src, so = tmp_path / "rt.c", tmp_path / "fakehip.so"
    src.write_text(RUNTIME)
    subprocess.run(["gcc", "-O1", "-w", "-fPIC", "-shared", str(src), "-o", str(so)], check=True)
    r = subprocess.run([sys.executable, "-c", PRELUDE + body, str(so), ROOT], capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


def test_failed_seeding_drops_the_self_norms_at_a_bandwidth(tmp_path):
    """The seeding works in the array that holds them."""
    _run(tmp_path, r"""
c, keep = ctx()
idx, xb, f = (C.c_int32 * 4)(0, 1, 2, 3), (C.c_float * (8 * 32))(), C.c_double()
L.check(lib.mbkk_init_centers(c, idx), c)
def sigma_launches():
    F.fake_launched(b"")
    L.check(lib.mbkk_objective_fwd(c, xb, 8, 1.5, None, C.byref(f)), c)
    return F.fake_launched(b"sigma")
first = sigma_launches()
assert first > 0, "the forward makes the self norms"
assert sigma_launches() == 0, "and keeps them"
F.fake_fail_d2d(1)
u = (C.c_double * 4)(0.1, 0.2, 0.3, 0.4)
assert lib.mbkk_init_kmeanspp(c, u, idx) == L.E_HIP
F.fake_fail_d2d(0)
assert sigma_launches() == first, "made anew after a seeding that failed"
""")
