"""Sources of the library's asynchronous copies, without a GPU: a stand-in for the HIP runtime that makes
every copy at the next synchronisation, the latest that the interface allows, and compares the source with
what it held when the copy was asked for.  Problems and a batch of two classes are driven through it (the
kernels do nothing); a source freed or changed too early is reported.
"""
import ctypes
import subprocess
import sys

STAND_IN = r"""
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
typedef struct op { struct op *next; void *dst; const void *src; void *was; size_t n; int host_src; } op;
static op *first, **tail = &first;
static int early, copies;
int stand_in_early(void) { return early; }
int stand_in_copies(void) { return copies; }
static void flush(void) {
    while (first) {
        op *o = first;
        if (o->host_src && memcmp(o->src, o->was, o->n)) early++;
        memmove(o->dst, o->was, o->n);
        first = o->next;
        free(o->was);
        free(o);
    }
    tail = &first;
}
int hipMemcpyAsync(void *dst, const void *src, size_t n, int kind, void *stream) {
    op *o = calloc(1, sizeof *o);
    if (kind != 1) flush();   /* a copy from the device's memory sees what was enqueued before it */
    o->dst = dst, o->src = src, o->n = n, o->host_src = kind == 1;
    o->was = malloc(n);
    memcpy(o->was, src, n);
    *tail = o, tail = &o->next;
    copies++;
    return 0;
}
int hipMemsetAsync(void *dst, int v, size_t n, void *s) { flush(); memset(dst, v, n); return 0; }
int hipMemcpy(void *dst, const void *src, size_t n, int kind) { flush(); memmove(dst, src, n); return 0; }
int hipStreamSynchronize(void *s) { flush(); return 0; }
int hipEventSynchronize(void *e) { flush(); return 0; }
int hipEventQuery(void *e) { flush(); return 0; }
int hipHostMalloc(void **p, size_t n, unsigned f) { *p = calloc(1, n); return 0; }
int hipHostFree(void *p) { free(p); return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipGetLastError(void) { return 0; }
const char *hipGetErrorString(int e) { return "stand-in"; }
int hipGetSymbolAddress(void **p, const void *s) { *p = 0; return 1; }
int hipLaunchKernel(const void *f, uint64_t gxy, uint32_t gz, uint64_t bxy, uint32_t bz, void **a, size_t l, void *s) { return 0; }
int hipEventCreate(void **e) { *e = malloc(1); return 0; }
int hipEventCreateWithFlags(void **e, unsigned f) { return hipEventCreate(e); }
int hipEventDestroy(void *e) { free(e); return 0; }
int hipEventRecord(void *e, void *s) { return 0; }
int hipEventElapsedTime(float *ms, void *a, void *b) { *ms = 0; return 0; }
int hipStreamCreateWithFlags(void **s, unsigned f) { *s = malloc(1); return 0; }
int hipStreamDestroy(void *s) { free(s); return 0; }
int hipStreamBeginCapture(void *s, int mode) { return 0; }
int hipStreamEndCapture(void *s, void **g) { *g = malloc(1); return 0; }
int hipGraphInstantiate(void **e, void *g, void *n, char *log, size_t size) { *e = malloc(1); return 0; }
int hipGraphLaunch(void *e, void *s) { return 0; }
int hipGraphDestroy(void *g) { free(g); return 0; }
int hipGraphExecDestroy(void *e) { free(e); return 0; }
int __hipPushCallConfiguration(uint64_t gxy, uint32_t gz, uint64_t bxy, uint32_t bz, size_t l, void *s) { return 0; }
int __hipPopCallConfiguration(void *g, void *b, size_t *l, void **s) { *l = 0; *s = 0; return 0; }
void **__hipRegisterFatBinary(const void *d) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **m) {}
void __hipRegisterFunction(void **m, const void *f, char *d, const char *n, unsigned t, void *a, void *b, void *c, void *e, int *w) {}
void __hipRegisterVar(void **m, void *v, char *d, char *n, int e, size_t s, int c, int g) {}
"""


def drive(stand_in_path):
    """Runs in a process of its own: the stand-in's symbols come before the HIP runtime's."""
    stand_in = ctypes.CDLL(stand_in_path, mode=ctypes.RTLD_GLOBAL)
    import numpy as np
    from paper_1406_7416_amd import adg, workloads as W
    L = adg.load()
    keep = []

    def workspace(nbytes):
        a = np.zeros(nbytes + 512, dtype=np.uint8)
        keep.append(a)
        return ctypes.c_void_p((a.ctypes.data + 255) & ~255)

    def problem(wl, mask=None):
        prm = adg._Params()
        prm.Ns, prm.limiter, prm.eps, prm.delta0 = 2 * wl.N + 1, 1, wl.eps, wl.delta0
        grid, h = adg._grid(wl), ctypes.c_void_p()
        adg._check(L.adg_create(ctypes.byref(grid), wl.N, wl.gamma, ctypes.byref(prm), ctypes.byref(h)))
        n = L.adg_workspace_bytes(h)
        adg._check(L.adg_bind(h, workspace(n), n, None))
        if mask is not None:
            adg._check(L.adg_set_mask(h, mask.ctypes.data_as(ctypes.POINTER(ctypes.c_uint8))))
        u, v = adg.project(wl, wl.N + 1)
        adg._check(L.adg_set_state(h, u.ctypes.data_as(ctypes.c_void_p), 0, adg._dp(v)))
        return h

    step = W.forward_facing_step(15, 5, 3)
    ps = [problem(W.explosion_2d(6, 3)), problem(step, W.step_mask(step).astype(np.uint8)),
          problem(W.explosion_2d(5, 2)), problem(W.explosion_2d(4, 3))]
    for h in ps:
        adg._check(L.adg_step(h, 1e-4))
        adg._check(L.adg_debug_poison(h, 0, 0, 1.0))
    b = ctypes.c_void_p()
    adg._check(L.adg_batch_create((ctypes.c_void_p * len(ps))(*[h.value for h in ps]), len(ps), ctypes.byref(b)))
    n = L.adg_batch_workspace_bytes(b)
    adg._check(L.adg_batch_bind(b, workspace(n), n, None))
    adg._check(L.adg_batch_step_cfl(b, 0.3, 3))
    adg._check(L.adg_batch_step_cfl(b, 0.2, 2))   # another CFL number: captured again
    L.adg_batch_destroy(b)
    for h in ps:
        L.adg_destroy(h)
    print("copies", stand_in.stand_in_copies(), "early", stand_in.stand_in_early())


def test_sources_live_until_the_copies_are_made(tmp_path):
    src, lib = tmp_path / "stand_in.c", tmp_path / "stand_in.so"
    src.write_text(STAND_IN)
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-w", str(src), "-o", str(lib)], check=True)
    out = subprocess.run([sys.executable, __file__, str(lib)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stderr[-2000:]
    words = out.stdout.split()
    assert int(words[1]) > 50 and int(words[3]) == 0, out.stdout


if __name__ == "__main__":
    import os
    sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    drive(sys.argv[1])
