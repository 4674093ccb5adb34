"""A double of the HIP runtime calls that libwpm.so makes, for host tests:
device memory is host memory, launches are recorded and not run.

`run(code)` runs Python code in a process of its own that has loaded the
double and then libwpm.so, and returns what it prints.  In it, `hip` is the
double: hip.launches() gives the launches so far as (kernel's symbol, grid,
block, dynamic LDS bytes, the bytes of each argument); the launch that clears
the outputs has no name.
"""
import os
import subprocess
import sys
import textwrap

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

SOURCE = r"""
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stdint.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;
typedef struct {
    char name[160];
    uint32_t grid, block;
    uint64_t lds, num_args;
    unsigned char args[8][256];
} launch_t;

enum { MOST = 256 };
static launch_t log_[MOST];
static int count_;
static dim3_t grid_, block_;
static size_t lds_;
static void *stream_;

int stub_count(void) { return count_; }
launch_t *stub_launch(int i) { return &log_[i]; }

int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t lds, void *st) {
    grid_ = g; block_ = b; lds_ = lds; stream_ = st;
    return 0;
}
int __hipPopCallConfiguration(dim3_t *g, dim3_t *b, size_t *lds, void **st) {
    *g = grid_; *b = block_; *lds = lds_; *st = stream_;
    return 0;
}
// (the kernels of other names that these tests reach: clear_outputs)
static int args_of(const char *name) { return strstr(name, "_kernel") ? 4 : 6; }
int hipLaunchKernel(const void *f, dim3_t g, dim3_t b, void **args, size_t lds, void *st) {
    Dl_info info;
    (void)st;
    if (count_ >= MOST) return 1;
    launch_t *l = &log_[count_++];
    memset(l, 0, sizeof *l);
    if (dladdr(f, &info) && info.dli_sname && info.dli_saddr == f) strncpy(l->name, info.dli_sname, sizeof l->name - 1);
    l->grid = g.x; l->block = b.x; l->lds = lds;
    l->num_args = args_of(l->name);
    for (uint64_t i = 0; i < l->num_args; ++i) memcpy(l->args[i], args[i], l->num_args == 4 && i == 3 ? 120 : 8);
    return 0;
}
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int attr, int dev) { (void)attr; (void)dev; *v = 65536; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int b, size_t lds) {
    (void)f; (void)b; (void)lds;
    *n = 1;
    return 0;
}
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *st) {
    (void)kind; (void)st;
    memcpy(d, s, n);
    return 0;
}
int hipStreamSynchronize(void *st) { (void)st; return 0; }
int hipPointerGetAttributes(void *a, const void *p) { (void)a; (void)p; return 1; }
int hipGetLastError(void) { return 0; }
static uint64_t scratch_[4096];
int hipGetSymbolAddress(void **p, const void *sym) { (void)sym; *p = scratch_; return 0; }
"""

PRELUDE = r"""
import ctypes, os, sys
sys.path.insert(0, {root!r})
_so = ctypes.CDLL({so!r}, mode=ctypes.RTLD_GLOBAL)  # found before the runtime's own

class Launch(ctypes.Structure):
    _fields_ = [("name", ctypes.c_char * 160), ("grid", ctypes.c_uint32), ("block", ctypes.c_uint32),
                ("lds", ctypes.c_uint64), ("num_args", ctypes.c_uint64),
                ("args", (ctypes.c_ubyte * 256) * 8)]

class hip:
    @staticmethod
    def launches():
        _so.stub_launch.restype = ctypes.POINTER(Launch)
        out = []
        for i in range(_so.stub_count()):
            l = _so.stub_launch(i).contents
            out.append((l.name.decode(), l.grid, l.block, l.lds, [bytes(l.args[j]) for j in range(l.num_args)]))
        return out

import numpy as np
from paper_2301_00806_amd import _lib as L, engine as E
"""


def build(folder) -> str:
    src, so = os.path.join(str(folder), "hipdouble.c"), os.path.join(str(folder), "libhipdouble.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", so, src, "-ldl"], check=True, capture_output=True)
    return so


def run(so: str, code: str, timeout: int = 120):
    """(exit status, stdout, stderr) of the code."""
    text = PRELUDE.format(root=ROOT, so=so) + textwrap.dedent(code)
    r = subprocess.run([sys.executable, "-c", text], capture_output=True, text=True, timeout=timeout, cwd=ROOT)
    return r.returncode, r.stdout, r.stderr
