"""A stand-in for the HIP runtime, for tests of the library's host path on a machine without a GPU.

``run(tmp_path, script)`` executes a Python script in a process of its own whose ``libdepo.so`` calls this
stand-in: device memory is host memory, copies are copies, kernels do nothing.  It keeps a log of the
kernels that would have run (the kernels of a captured graph once per replay), counts captures and replays,
and fails the captures it is told to.  The script has ``simulation(...)`` and ``fake`` (see PRELUDE)."""

import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
typedef struct { uint32_t x, y, z; } dim3;
#define OK 0
#define MAXK 4096
#define MAXLOG (1 << 20)
static const void *fn[MAXK]; static const char *name[MAXK]; static int n_fn;
static dim3 g_, b_; static size_t sh_; static void *st_;
/* kernels of the capture under way, of each graph, and of everything that ran */
typedef struct { int n; int k[MAXK]; } graph;
static graph *capturing;
static int *ran, n_ran, captures, instantiated, replays, fail_at = -1, events, ran_before[64];
int fake_captures(void) { return captures; }
int fake_replays(void) { return replays; }
int fake_ran(void) { return n_ran; }
/* kernels that had run when the k-th capture since the reset began */
int fake_ran_before_capture(int k) { return ran_before[k & 63]; }
const char *fake_name(int i) { return name[ran[i]]; }
void fake_reset(void) { n_ran = captures = replays = 0; fail_at = -1; }
/* the k-th capture from now on (0: the next) fails */
void fake_fail_capture(int k) { fail_at = captures + k; }
static void log_kernel(int k) {
  if (!ran) ran = malloc(MAXLOG * sizeof(int));
  if (capturing) { if (capturing->n < MAXK) capturing->k[capturing->n++] = k; }
  else if (n_ran < MAXLOG) ran[n_ran++] = k;
}
void **__hipRegisterFatBinary(const void *d) { static void *h[1]; (void)d; return h; }
void __hipUnregisterFatBinary(void **h) { (void)h; }
void __hipRegisterFunction(void **m, const void *f, char *d, const char *n, unsigned t, void *a, void *b, void *c, void *e, int *w) {
  (void)m; (void)d; (void)t; (void)a; (void)b; (void)c; (void)e; (void)w;
  if (n_fn < MAXK) { fn[n_fn] = f; name[n_fn++] = n; }
}
void __hipRegisterVar(void **m, void *v, char *h, char *n, int e, size_t s, int c, int g) {
  (void)m; (void)v; (void)h; (void)n; (void)e; (void)s; (void)c; (void)g;
}
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t sh, void *st) { g_ = g; b_ = b; sh_ = sh; st_ = st; return OK; }
int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *sh, void **st) { *g = g_; *b = b_; *sh = sh_; *st = st_; return OK; }
int hipLaunchKernel(const void *f, dim3 g, dim3 b, void **a, size_t sh, void *st) {
  (void)g; (void)b; (void)a; (void)sh; (void)st;
  for (int k = 0; k < n_fn; ++k) if (fn[k] == f) { log_kernel(k); return OK; }
  return 98;
}
static int last;
int hipGetLastError(void) { int e = last; last = OK; return e; }
const char *hipGetErrorString(int e) { return e ? "failed on request" : "no error"; }
int hipGetDevice(int *d) { *d = 0; return OK; }
int hipGetSymbolAddress(void **p, const void *s) { (void)s; *p = aligned_alloc(256, (size_t)64 << 20); return OK; }
static void *copy_at; static size_t copy_bytes;
/* the last synchronous copy */
void *fake_copy_at(void) { return copy_at; }
size_t fake_copy_bytes(void) { return copy_bytes; }
int hipMemcpy(void *d, const void *s, size_t n, int k) { (void)k; copy_at = d; copy_bytes = n; memcpy(d, s, n); return OK; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st) { (void)k; (void)st; memcpy(d, s, n); return OK; }
int hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = malloc(1); return OK; }
int hipStreamDestroy(void *s) { free(s); return OK; }
int hipStreamSynchronize(void *s) { (void)s; return OK; }
int hipStreamWaitEvent(void *s, void *e, unsigned f) { (void)s; (void)e; (void)f; return OK; }
int hipEventCreate(void **e) { *e = malloc(1); ++events; return OK; }
int hipEventCreateWithFlags(void **e, unsigned f) { (void)f; return hipEventCreate(e); }
int hipEventDestroy(void *e) { free(e); --events; return OK; }
int hipEventRecord(void *e, void *s) { (void)e; (void)s; return OK; }
int hipEventElapsedTime(float *ms, void *a, void *b) { (void)a; (void)b; *ms = 1.0f; return OK; }
int hipStreamBeginCapture(void *s, int mode) {
  (void)s; (void)mode;
  ran_before[captures & 63] = n_ran;
  if (captures++ == fail_at) return last = 1;
  capturing = calloc(1, sizeof(graph));
  return OK;
}
int hipStreamEndCapture(void *s, void **g) {
  (void)s;
  *g = capturing;
  capturing = 0;
  return *g ? OK : 1;
}
int hipGraphInstantiate(void **x, void *g, void *n, char *l, size_t z) {
  (void)n; (void)l; (void)z;
  *x = malloc(sizeof(graph));
  memcpy(*x, g, sizeof(graph));
  ++instantiated;
  return OK;
}
int hipGraphDestroy(void *g) { free(g); return OK; }
int hipGraphExecDestroy(void *x) { free(x); --instantiated; return OK; }
int hipGraphLaunch(void *x, void *s) {
  (void)s;
  graph *g = x;
  ++replays;
  for (int i = 0; i < g->n; ++i) log_kernel(g->k[i]);
  return OK;
}
"""

PRELUDE = r'''
import ctypes as C, json, sys
import numpy as np
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)      # before the library, whose HIP calls then come here
fake.fake_name.restype = C.c_char_p
from paper_2205_04979_amd import depo
from synthetic.workloads import physical_params
R, L = 0.01, 0.04

def simulation(sizes, real_bytes=4, p3m=None, reorder=0, cfg=None, graph=True, **params):
    """A seeded context over samples of these sizes; its ``step(n)`` returns the status."""
    p = physical_params(180.0, **params)
    ctx = depo.Context(p, real_bytes)
    lib, h = ctx._L, ctx._h
    if p3m:
        ctx.check(lib.depo_set_p3m(h, *p3m), "p3m")
    ctx.set_layout(np.concatenate([[0], np.cumsum(sizes)]), 4, 4, 4)
    ctx.work = np.zeros(ctx.workspace_bytes() + 256, np.uint8)
    at = (ctx.work.ctypes.data + 255) // 256 * 256
    ctx.check(lib.depo_bind(h, at, ctx.workspace_bytes()), "bind")
    f = np.zeros((4, 4, 4, 3))
    ctx.check(lib.depo_init_field(h, depo._dptr(f), None), "field")
    if cfg:
        ctx.check(lib.depo_set_kernel_config(h, *cfg, int(graph)), "shape")
    ctx.check(lib.depo_set_reorder(h, reorder), "reorder")
    n = int(sum(sizes))
    rng = np.random.default_rng(1)
    x = rng.uniform(-0.6 * R, 0.6 * R, (n, 3))
    x[:, 0] = rng.uniform(0, L, n)
    ctx.x, ctx.d, ctx.q = x, np.full(n, 1e-5), 1e-15 * rng.normal(size=n)
    ctx.sp = (depo.SampleParams * len(sizes))(*[depo.SampleParams(1.0, 1e-20, 300.0) for _ in sizes])
    def seed():
        ctx.check(lib.depo_seed(h, ctx.sp, depo._dptr(ctx.x), None, depo._dptr(ctx.d), depo._dptr(ctx.q), None), "seed")
    ctx.seed = seed
    ctx.step = lambda k: lib.depo_step(h, k, None)
    def steps_done():
        t = (depo.Tally * len(sizes))()
        ctx.check(lib.depo_tally_read(h, t, None), "tally")
        return round(t[0].t / p["dt"])
    ctx.steps_done = steps_done
    seed()
    return ctx

fake.fake_copy_at.restype = C.c_void_p
fake.fake_copy_bytes.restype = C.c_size_t

def items(ctx, *cfg):
    """The work items of the symmetric pair kernel in a shape (the call's last copy): target, number of targets, source,
    number of sources, sample, diagonal."""
    ctx.check(ctx._L.depo_set_kernel_config(ctx._h, *cfg, 64, 2, 1), "shape")
    n = fake.fake_copy_bytes() // 4
    return np.ctypeslib.as_array(C.cast(fake.fake_copy_at(), C.POINTER(C.c_int32)), (n,)).reshape(-1, 8)[:, :6].copy()

def adjoint(ctx, steps=2, ckpt=1):
    """Names of the kernels of a gradient."""
    size = C.c_size_t()
    ctx.check(ctx._L.depo_adjoint_workspace_bytes(ctx._h, steps, ckpt, C.byref(size)), "size")
    work = np.zeros(size.value + 256, np.uint8)
    s = len(ctx.sp)
    w, g = np.ones(s), np.zeros((s, 3))
    fake.fake_reset()
    ctx.check(ctx._L.depo_adjoint(ctx._h, steps, ckpt, depo._dptr(w), depo._dptr(g), (work.ctypes.data + 255) // 256 * 256,
                                  size.value, None), "adjoint")
    return ran()

def ran():
    """Names of the kernels that ran since the last reset, in order."""
    return [fake.fake_name(i).decode() for i in range(fake.fake_ran())]

def steps_run():
    """Steps among them: each one ends in one k_finish or k_finish_prepare."""
    return sum("k_finish" in k for k in ran())
'''


def run(tmp_path, script: str):
    """The JSON that the script prints last."""
    src, so = tmp_path / "fake_hip.c", tmp_path / "libfake_hip.so"
    src.write_text(SOURCE)
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", str(src), "-o", str(so)], check=True)
    r = subprocess.run([sys.executable, "-c", PRELUDE + script, str(so)], capture_output=True, text=True, cwd=ROOT,
                       timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    return json.loads(r.stdout.splitlines()[-1])
