"""A stand-in for the HIP runtime, for host-side tests of liblbw.so on the CPU.

It defines the runtime functions the library calls between a step or a reduction
and the device, does nothing on any device, and keeps a log: one line per kernel
launch (name, grid, block, dynamic LDS, last argument as a pointer), wait, graph
and pinned allocation.  `run` compiles it, loads it ahead of the library in a
fresh interpreter, so that the library binds to it, and runs a script there with
these names: `lib` (the bound library), `lbw` (the package's binding), `handle`
(a run over made-up device addresses) and `log` (the lines since the last call).
Errors are set from the script: `fake.fake_last_error(e)` is what the next
hipGetLastError returns, `fake.fake_sync_error(e)` what waits return from then on.
"""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#define _GNU_SOURCE
#include <stdarg.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
typedef int err;
typedef struct { uint32_t x, y, z; } dim3;
typedef void *stream;
static char text[1 << 22];
static size_t used;
static void note(const char *fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    used += (size_t)vsnprintf(text + used, sizeof text - used, fmt, ap);
    va_end(ap);
}
const char *fake_log(void) { return text; }
void fake_clear(void) { used = 0; text[0] = 0; }
static err last_error, sync_error;
static int mode, graphs;
void fake_last_error(err e) { last_error = e; }
void fake_sync_error(err e) { sync_error = e; }

/* kernel registration: host stub address -> device name, number of arguments unknown */
static struct { const void *f; char name[512]; } kernel[8192];
static int kernels;
static int handle_;
void **__hipRegisterFatBinary(const void *d) { (void)d; return (void **)&handle_; }
void __hipUnregisterFatBinary(void **h) { (void)h; }
void __hipRegisterFunction(void **h, const void *f, char *df, const char *name, unsigned n, void *a, void *b,
                           void *c, void *d, int *e) {
    (void)h; (void)df; (void)n; (void)a; (void)b; (void)c; (void)d; (void)e;
    kernel[kernels].f = f;
    snprintf(kernel[kernels++].name, 512, "%s", name);
}
void __hipRegisterVar(void **h, void *v, char *hv, char *dv, int e, size_t s, int c, int g) {
    (void)h; (void)v; (void)hv; (void)dv; (void)e; (void)s; (void)c; (void)g;
}
static struct { dim3 g, b; size_t lds; stream s; } conf;
err __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, stream s) {
    conf.g = g; conf.b = b; conf.lds = lds; conf.s = s;
    return 0;
}
err __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, stream *s) {
    *g = conf.g; *b = conf.b; *lds = conf.lds; *s = conf.s;
    return 0;
}
err hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t lds, stream s) {
    const char *name = "?";
    (void)s;
    for (int i = 0; i < kernels; ++i) if (kernel[i].f == f) name = kernel[i].name;
    /* the reductions' first pass: argument 6 is where the partials go */
    void *to = strstr(name, "k_partial") ? *(void **)args[6] : NULL;
    note("launch %s %u %u %u %u %zu %p\n", name, g.x, g.y, g.z, b.x, lds, to);
    return 0;
}
err hipGetLastError(void) { const err e = last_error; last_error = 0; return e; }
const char *hipGetErrorString(err e) { (void)e; return "made-up error"; }
err hipStreamSynchronize(stream s) { (void)s; note("wait %d\n", sync_error); return sync_error; }
err hipMemcpyAsync(void *d, const void *s, size_t n, int k, stream st) {
    (void)d; (void)s; (void)k; (void)st;
    note("copy %zu\n", n);
    return 0;
}
err hipThreadExchangeStreamCaptureMode(int *m) { const int t = mode; mode = *m; *m = t; return 0; }
err hipHostMalloc(void **p, size_t n, unsigned f) {
    (void)f;
    note("pinned %zu mode %d\n", n, mode);
    *p = calloc(1, n);
    return *p ? 0 : 2;
}
err hipHostGetDevicePointer(void **d, void *h, unsigned f) { (void)f; *d = h; return 0; }
err hipGetDevice(int *d) { *d = 0; return 0; }
err hipDeviceGetAttribute(int *v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
err hipStreamBeginCapture(stream s, int m) { (void)s; (void)m; note("capture\n"); return 0; }
err hipStreamEndCapture(stream s, void **g) { (void)s; *g = (void *)(uintptr_t)++graphs; return 0; }
err hipGraphInstantiate(void **e, void *g, void *a, char *b, size_t n) {
    (void)a; (void)b; (void)n;
    *e = g;
    note("instantiate %p\n", g);
    return 0;
}
err hipGraphLaunch(void *e, stream s) { (void)s; note("replay %p\n", e); return 0; }
err hipGraphExecDestroy(void *e) { note("destroy %p\n", e); return 0; }
err hipGraphDestroy(void *g) { (void)g; return 0; }
"""

PRELUDE = r"""
import ctypes, sys
sys.path.insert(0, {root!r})
fake = ctypes.CDLL({so!r}, mode=ctypes.RTLD_GLOBAL)
fake.fake_log.restype = ctypes.c_char_p
from paper_2106_07694_amd import lbw
lib = lbw.load()

def handle(cfgs, stream=0x7000, scratch=1 << 24, **launch):
    cfgs = [cfgs] if isinstance(cfgs, lbw.RunConfig) else cfgs
    bufs = (lbw.CBuffers * len(cfgs))()
    for b in bufs:
        for i, k in enumerate(("f", "c", "c_s1", "c_s2", "s", "s_tmp", "u", "deposit", "scratch")):
            setattr(b, k, (i + 1) << 40)
        b.scratch_bytes = scratch
    h = ctypes.c_void_p()
    lbw.check(lib.lbw_create((lbw.CConfig * len(cfgs))(*[c.to_c() for c in cfgs]), bufs, len(cfgs),
                             ctypes.c_void_p(stream), ctypes.byref(h)))
    if launch:
        l = lbw.CLaunch(**launch)
        lbw.check(lib.lbw_set_launch(h, ctypes.byref(l)))
    log()
    return h

def log():
    lines = fake.fake_log().decode().splitlines()
    fake.fake_clear()
    return lines

def launches(part):
    '''(grid, block, dynamic LDS) of the launches of kernels whose name holds `part`.'''
    out = []
    for l in log():
        w = l.split()
        if w[0] == "launch" and part in w[1]:
            out.append(((int(w[2]), int(w[3]), int(w[4])), int(w[5]), int(w[6])))
    return out
"""


def run(tmp_path, script):
    """Run `script` after the prelude; it must end by itself with status 0."""
    src, so = str(tmp_path / "fake_hip.c"), str(tmp_path / "fake_hip.so")
    with open(src, "w") as fh:
        fh.write(SOURCE)
    subprocess.run(["gcc", "-std=c11", "-O1", "-Wall", "-shared", "-fPIC", src, "-o", so], check=True)
    r = subprocess.run([sys.executable, "-c", PRELUDE.format(root=ROOT, so=so) + script], capture_output=True,
                       text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout
