"""A stand-in for the HIP runtime, for host logic without a GPU: memory is host
memory, kernels do nothing, a launch can be made to fail, and the names of the
launched kernels are kept.  `run` executes a script in a process of its own that
loads the stand-in ahead of the library, with `hip` (ctypes), `launched()` (the
kernels' names since the last call) and `lpt` defined."""
import os
import subprocess
import sys

from paper_2607_17836_amd import lpt

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <stdlib.h>
#include <string.h>
typedef int E;
#define MAXK 4096
static const void *host_fn[MAXK];
static char *name[MAXK];
static int nk = 0, left = -1, last = 0, nl = 0;
static const char *seen[MAXK];
void stand_in_fail_after(int launches) { left = launches; }
int stand_in_launches(void) { return nl; }
const char *stand_in_launch(int k) { return seen[k]; }
void stand_in_reset(void) { nl = 0; }
void __hipRegisterFunction(void **m, const void *f, char *dev, const char *dn)
{ if (nk < MAXK) { host_fn[nk] = f; name[nk++] = strdup(dn); } }
E hipLaunchKernel(const void *f)
{
    int k;
    if (left == 0) return last = 1;
    if (left > 0) --left;
    for (k = 0; k < nk && host_fn[k] != f; ++k) {}
    if (nl < MAXK) seen[nl++] = k < nk ? name[k] : "?";
    return 0;
}
E hipGetLastError() { int e = last; last = 0; return e; }
const char *hipGetErrorString(E e) { return e ? "refused" : "ok"; }
static int mallocs = 0;
int stand_in_mallocs(void) { int m = mallocs; mallocs = 0; return m; }
E hipMalloc(void **p, size_t n) { ++mallocs; *p = calloc(1, n); return *p ? 0 : 2; }
E hipFree(void *p) { free(p); return 0; }
E hipMemcpyAsync(void *d, const void *s, size_t n) { memcpy(d, s, n); return 0; }
E hipMemsetAsync(void *d, int v, size_t n) { return 0; }
E hipGetDevice(int *d) { *d = 0; return 0; }
E hipSetDevice(int d) { return 0; }
E hipStreamSynchronize(void *s) { return 0; }
E hipDeviceGetAttribute(int *v) { *v = 256; return 0; }
E hipFuncGetAttributes(void *a) { memset(a, 0, 56); return 0; }
E hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n) { *n = 4; return 0; }
E hipGetSymbolAddress(void **p, const void *s) { static char here[256]; *p = here; return 0; }
E __hipPushCallConfiguration() { return 0; }
E __hipPopCallConfiguration(unsigned *g, unsigned *b, size_t *n, void **s)
{ g[0] = g[1] = g[2] = b[0] = b[1] = b[2] = 1; *n = 0; *s = 0; return 0; }
void **__hipRegisterFatBinary() { static void *h; return &h; }
void __hipRegisterVar() {}
void __hipUnregisterFatBinary() {}
"""

HEAD = r"""
import ctypes, sys
hip = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
hip.stand_in_launch.restype = ctypes.c_char_p
sys.modules["torch"] = None   # whose HIP runtime would come with it
import numpy as np
from paper_2607_17836_amd import lpt

def launched():
    out = [hip.stand_in_launch(k).decode() for k in range(hip.stand_in_launches())]
    hip.stand_in_reset()
    return out
"""


def run(script, tmp_path, *args):
    """The script's standard output; its arguments are sys.argv[2:]."""
    if not os.path.exists(lpt.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    src, so = os.path.join(tmp_path, "hip.c"), os.path.join(tmp_path, "libhip_stand_in.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run(["gcc", "-w", "-shared", "-fPIC", "-o", so, src], check=True)
    r = subprocess.run([sys.executable, "-c", HEAD + script, so, *map(str, args)], cwd=ROOT,
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout
