"""Host code of the library without a GPU: a stand-in for the HIP runtime, compiled here and loaded in front of it in a process of its
own, that writes down what the library asks and launches.  A call's pointers are numbers that nothing follows.

The stand-in has 256 compute units of 160 KB of LDS and, like the runtime, takes more than 64 KB of dynamic LDS only for a kernel whose
attribute says so."""
import json
import os
import subprocess
import sys

import debug_lib

SOURCE = r"""
#include <stdint.h>
#include <stdio.h>
#include <string.h>
typedef struct { uint32_t x, y, z; } dim3;
static struct { const void *fn; char name[256]; int lds; } kernels[256];
static int n_kernels;
static struct { dim3 grid, block; size_t lds; void *stream; } pushed;
static FILE *out;
static int kernel(const void *fn)
{
    for (int i = 0; i < n_kernels; ++i)
        if (kernels[i].fn == fn)
            return i;
    return -1;
}
void fake_log(const char *path) { out = fopen(path, "w"); }
void fake_flush(void) { fflush(out); }
void **__hipRegisterFatBinary(const void *d) { static void *h; (void)d; return &h; }
void __hipUnregisterFatBinary(void **h) { (void)h; }
void __hipRegisterFunction(void **m, const void *fn, char *d, const char *name, unsigned n, void *a, void *b, void *c, void *e, int *w)
{
    if (n_kernels < 256) {
        kernels[n_kernels].fn = fn;
        strncpy(kernels[n_kernels++].name, name, 255);
    }
}
void __hipRegisterVar(void **m, void *v, char *h, char *d, int e, size_t s, int c, int g) {}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void *stream)
{
    pushed.grid = grid, pushed.block = block, pushed.lds = lds, pushed.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, void **stream)
{
    *grid = pushed.grid, *block = pushed.block, *lds = pushed.lds, *stream = pushed.stream;
    return 0;
}
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipGetLastError(void) { return 0; }
int hipDeviceGetAttribute(int *v, int a, int d) { *v = 256; return 0; }
int hipGetSymbolAddress(void **p, const void *s) { *p = (void *)4096; return 0; }
int hipFuncSetAttribute(const void *fn, int attr, int v)
{
    kernels[kernel(fn)].lds = v;
    return 0;
}
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *fn, int threads, size_t lds)
{
    const int k = kernel(fn), ok = lds <= 65536 || (int)lds <= kernels[k].lds;
    *n = ok ? 163840 / (int)lds : 0;
    fprintf(out, "{\"what\": \"occupancy\", \"kernel\": \"%s\", \"allowed\": %d, \"fits\": %d}\n", kernels[k].name, ok, *n);
    return ok ? 0 : 1;
}
int hipLaunchKernel(const void *fn, dim3 grid, dim3 block, void **args, size_t lds, void *stream)
{
    const int k = kernel(fn), ok = lds <= 65536 || (int)lds <= kernels[k].lds;
    fprintf(out, "{\"what\": \"launch\", \"kernel\": \"%s\", \"grid\": %u, \"threads\": %u, \"allowed\": %d", kernels[k].name, grid.x, block.x, ok);
    if (strstr(kernels[k].name, "planned")) {   // (the plan: 417 words)
        const uint32_t *w = (const uint32_t *)args[1];
        fprintf(out, ", \"plan\": [%u", w[0]);
        for (int i = 1; i < 417; ++i)
            fprintf(out, ", %u", w[i]);
        fprintf(out, "]");
    }
    fprintf(out, "}\n");
    return ok ? 0 : 1;
}
"""

RUN = r"""
import ctypes, json, sys
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
fake.fake_log(sys.argv[3].encode())
lib = ctypes.CDLL(sys.argv[2])
out = []
for heads, s_q, s_kv, d, causal, f16, tiling in json.loads(sys.argv[4]):
    f = lib.attn_bwd_tiling if tiling else lib.attn_bwd_f16 if f16 else lib.attn_bwd
    p, i = ctypes.c_void_p, ctypes.c_int
    x = [4096 * (n + 1) for n in range(10)]
    if tiling:
        f.argtypes = [p] * 10 + [i] * 6 + [ctypes.c_float, p, i]
        rc = f(*x, 1, heads, s_q, s_kv, f16, causal, 0.1, None, tiling)
    else:
        f.argtypes = [p] * 10 + [i] * 6 + [ctypes.c_float, p]
        rc = f(*x, 1, heads, s_q, s_kv, d, causal, 0.1, None)
    fake.fake_flush()
    out.append((rc, sum(1 for _ in open(sys.argv[3]))))
print(json.dumps(out))
"""


def backward_calls(tmp_path, calls):
    """What each of `calls` -- (heads, S_q, S_kv, D, causal, f16, tiling or 0) -- returns, and the lines it leaves."""
    c, so, log = (str(tmp_path / n) for n in ("fake_hip.c", "fake_hip.so", "log"))
    with open(c, "w") as f:
        f.write(SOURCE)
    subprocess.run([os.environ.get("CC", "gcc"), "-O1", "-shared", "-fPIC", "-w", "-o", so, c], check=True)
    done = subprocess.run([sys.executable, "-c", RUN, so, debug_lib.PATH, log, json.dumps(calls)], check=True, stdout=subprocess.PIPE)
    lines, out, at = [json.loads(x) for x in open(log)], [], 0
    for rc, n in json.loads(done.stdout.splitlines()[-1]):
        out.append((rc, lines[at:n]))
        at = n
    return out
