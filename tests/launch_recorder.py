"""What a call launches, without a GPU: the library is loaded in a child process behind a stand-in for the sixteen functions of the HIP runtime that it calls, which keeps every launch
(kernel, grid, threads, dynamic LDS) and every look-up of a device variable instead of carrying it out.  Tensors are addresses that nobody reads."""
import ctypes
import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
INT, INT64, FLOAT, POINTER, SIZE, QPARAMS = "i", "q", "f", "p", "z", "Q"

STUB = r"""
#include <stdio.h>
#include <stdlib.h>
#include <stddef.h>
typedef struct { unsigned x, y, z; } dim3;
static struct { const void *host; const char *name; } kernels[4096];
static int n_kernels;
static dim3 grid_, block_;
static size_t lds_;
static void *stream_, *none;
static char page[4096];
void **__hipRegisterFatBinary(const void *data) { return &none; }
void __hipUnregisterFatBinary(void **m) {}
void __hipRegisterFunction(void **m, const void *host, char *dev, const char *name, unsigned limit, void *tid, void *bid, dim3 *b, dim3 *g, int *w)
{
    if (n_kernels == 4096) abort();
    kernels[n_kernels].host = host;
    kernels[n_kernels++].name = name;
}
void __hipRegisterVar(void **m, void *var, char *host, char *dev, int ext, size_t size, int constant, int global) {}
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, void *stream) { grid_ = g; block_ = b; lds_ = lds; stream_ = stream; return 0; }
int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, void **stream) { *g = grid_; *b = block_; *lds = lds_; *stream = stream_; return 0; }
int hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t lds, void *stream)
{
    const char *name = "?";
    for (int i = 0; i < n_kernels; ++i)
        if (kernels[i].host == f) name = kernels[i].name;
    printf("launch %s %u %u %u %u %zu\n", name, g.x, g.y, g.z, b.x * b.y * b.z, lds);
    return 0;
}
int hipGetSymbolAddress(void **p, const void *symbol) { printf("symbol\n"); *p = page; return 0; }
int hipDeviceGetAttribute(int *v, int attribute, int device) { *v = 256; return 0; }
int hipFuncSetAttribute(const void *f, int attribute, int value) { return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipGetLastError(void) { return 0; }
int hipEventCreate(void **e) { *e = page; return 0; }
int hipEventRecord(void *e, void *stream) { return 0; }
int hipEventSynchronize(void *e) { return 0; }
int hipEventElapsedTime(float *ms, void *a, void *b) { *ms = 0.0f; return 0; }
void recorder_next(int call) { printf("call %d\n", call); fflush(stdout); }
void recorder_end(int call, int status) { printf("status %d\n", status); fflush(stdout); }
"""

CHILD = r"""
import ctypes, json, sys
stub = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)      # (before the library and the runtime that it names: their symbols are found here first)
lib = ctypes.CDLL(sys.argv[2])
class QParams(ctypes.Structure):
    _fields_ = [("lo", ctypes.c_int32), ("n_levels", ctypes.c_int32), ("delta", ctypes.c_float), ("alpha", ctypes.c_float), ("top_k", ctypes.c_int32)]
types = {"i": ctypes.c_int32, "q": ctypes.c_int64, "f": ctypes.c_float, "p": ctypes.c_void_p, "z": ctypes.c_size_t}
for number, (name, args) in enumerate(json.load(sys.stdin)):
    stub.recorder_next(number)
    status = getattr(lib, name)(*(ctypes.byref(QParams(*v)) if t == "Q" else types[t](v) for t, v in args))
    stub.recorder_end(number, status)
"""

A = 1 << 32      # an aligned address


class Launch:
    def __init__(self, name, fields):
        self.name = name                                   # demangled, with its template arguments
        self.grid, self.threads, self.lds = tuple(int(v) for v in fields[:3]), int(fields[3]), int(fields[4])

    def __repr__(self):
        return "%s %s %d %d" % (self.name, self.grid, self.threads, self.lds)


def record(tmp_path, calls):
    """[(entry point, [(type, value)])] -> for every call its launches and how many device variables it looked up."""
    import paper_2501_09849_amd.build as build
    if not os.path.exists(build.LIB_PATH):
        build.build_lib()
    source, stub = tmp_path / "stub.c", tmp_path / "stub.so"
    source.write_text(STUB)
    subprocess.run(["g++", "-x", "c", "-O1", "-w", "-shared", "-fPIC", str(source), "-o", str(stub)], check=True)
    out = subprocess.run([sys.executable, "-c", CHILD, str(stub), build.LIB_PATH], input=json.dumps(calls), capture_output=True, text=True, check=True).stdout
    out = subprocess.run(["c++filt"], input=out, capture_output=True, text=True, check=True).stdout
    seen = []
    for line in out.splitlines():
        kind, _, rest = line.partition(" ")
        if kind == "call":
            seen.append(([], 0))
        elif kind == "launch":
            name, *fields = rest.rsplit(" ", 5)
            seen[-1][0].append(Launch(name, fields))
        elif kind == "symbol":
            seen[-1] = (seen[-1][0], seen[-1][1] + 1)
        elif kind == "status":
            assert rest == "0", (calls[len(seen) - 1], rest)
    assert len(seen) == len(calls)
    return seen


def _size(name, *args):
    import paper_2501_09849_amd as cdl
    return getattr(cdl, name)(*args)


def conv_fwd(B, H, W, C, N, R, S, stride, pad, x_offset=0):
    return ("cdl_qconv_fwd", [(POINTER, A), (POINTER, A)] + [(INT, v) for v in (B, H, W, C, N, R, S, stride, pad)] + [(FLOAT, 0.5), (FLOAT, 0.25), (INT, x_offset), (POINTER, None),
            (POINTER, A), (POINTER, A), (SIZE, 256 + (N * 4 + 255) // 256 * 256), (POINTER, None)])


def gemm_fwd(M, N, K):
    return ("cdl_qgemm_fwd", [(POINTER, A), (POINTER, A), (INT, M), (INT, N), (INT, K), (FLOAT, 0.5), (FLOAT, 0.25), (POINTER, None), (POINTER, A), (POINTER, A), (SIZE, 1 << 40), (POINTER, None)])


RINGS = {"RingShape<2, 4, 4, 2, 5, 1>": "wide", "RingShape<2, 2, 4, 2, 3, 2>": "tall", "RingShape<4, 1, 2, 2, 4, 2>": "narrow", "RingShape<2, 2, 2, 2, 5, 2>": "square", "RingShape<4, 1, 1, 2, 6, 2>": "low"}


def tile_form(launches):
    """Of a forward product: the tiles with direct loads (256 x 256, 256 x 128, 256 x 64, 128 x 128, 128 x 64), or staged ones, or another kernel."""
    names = [l.name for l in launches if "dma_kernel" in l.name]
    if names:
        return next(form for shape, form in RINGS.items() if shape in names[0])
    return "staged" if any("::qgemm_kernel<" in l.name or "::qconv_kernel<" in l.name for l in launches) else "other"


def gemm_bwd(M, N, K, want, b_offset=0):
    """want: a, b or both"""
    return ("cdl_qgemm_bwd_offset", [(POINTER, A), (POINTER, A), (POINTER, A), (INT, M), (INT, N), (INT, K), (FLOAT, 0.5), (FLOAT, 0.25), (INT, 0), (INT, b_offset), (POINTER, A if want != "b" else None),
            (POINTER, A if want != "a" else None), (POINTER, A), (SIZE, 1 << 40), (POINTER, None)])


def conv_bwd_weights(B, H, W, C, N, R, S, stride, pad, x_offset=0):
    return ("cdl_qconv_bwd_weights", [(POINTER, A), (POINTER, A)] + [(INT, v) for v in (B, H, W, C, N, R, S, stride, pad)] + [(FLOAT, 0.5), (INT, x_offset), (POINTER, A), (POINTER, A), (SIZE, 1 << 40), (POINTER, None)])
