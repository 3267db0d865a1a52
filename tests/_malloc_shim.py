"""A process whose device allocations are counted and can be made to fail:
a small library with a hipMalloc and hipFree of its own, loaded before
liblbm2p.so so that the calls of liblbm2p.so reach it.  Import this module
only in a process that has not loaded liblbm2p.so yet (see
test_gpu_memory.py)."""
import ctypes as C
import os
import subprocess
import tempfile

SOURCE = r"""
#include <dlfcn.h>
#include <stddef.h>
typedef int (*malloc_t)(void **, size_t);
typedef int (*free_t)(void *);
static malloc_t real_malloc;
static free_t real_free;
static struct { void *p; size_t n; } held[1 << 16];
long shim_calls, shim_fail = -1;   /* call number shim_fail finds no memory */
size_t shim_live;
int shim_init(const char *runtime) {
    void *h = dlopen(runtime, RTLD_NOW | RTLD_LOCAL);
    if (!h) return 1;
    real_malloc = (malloc_t)dlsym(h, "hipMalloc");
    real_free = (free_t)dlsym(h, "hipFree");
    return !real_malloc || !real_free;
}
int hipMalloc(void **p, size_t n) {
    if (shim_calls++ == shim_fail) {
        *p = NULL;
        return 2; /* hipErrorOutOfMemory */
    }
    int rc = real_malloc(p, n);
    if (rc) return rc;
    for (int i = 0; i < 1 << 16; ++i)
        if (!held[i].p) {
            held[i].p = *p;
            held[i].n = n;
            break;
        }
    shim_live += n;
    return 0;
}
int hipFree(void *p) {
    for (int i = 0; p && i < 1 << 16; ++i)
        if (held[i].p == p) {
            shim_live -= held[i].n;
            held[i].p = NULL;
            break;
        }
    return real_free(p);
}
"""


class Shim:
    def __init__(self):
        with tempfile.TemporaryDirectory() as d:
            src, so = os.path.join(d, "shim.c"), os.path.join(d, "shim.so")
            with open(src, "w") as f:
                f.write(SOURCE)
            subprocess.run(["gcc", "-O1", "-fPIC", "-shared", "-o", so, src, "-ldl"], check=True)
            self.lib = C.CDLL(so, mode=C.RTLD_GLOBAL)
        from paper_1908_09235_amd import lbm
        lbm.lib()
        assert self.lib.shim_init(b"libamdhip64.so.7") == 0

    def _var(self, name, kind):
        return kind.in_dll(self.lib, name)

    def start(self, fail=-1):
        """Counts from here; allocation number `fail` finds no memory."""
        self._var("shim_calls", C.c_long).value = 0
        self._var("shim_fail", C.c_long).value = fail

    @property
    def calls(self):
        return self._var("shim_calls", C.c_long).value

    @property
    def live(self):
        return self._var("shim_live", C.c_size_t).value
