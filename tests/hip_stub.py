"""The library's host code without a GPU: a stub of the HIP runtime calls that
gd_create and an apply make, loaded ahead of the runtime in a child process, which records
allocations and launches in place of making them.  Tests pass child code that
uses the names below; kernels never run, so pointers may hold anything."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1704_05021_amd", "libgd.so")

STUB = r"""
#include <stddef.h>
#include <stdint.h>
typedef struct { uint32_t x, y, z; } dim3_t;
int g_launches, g_allocs, g_frees, g_captured_stream, g_other_capture, g_refused, g_mode;
uintptr_t g_last_alloc, g_last_free, g_next = 0x10000000;
size_t g_last_size, g_total;
dim3_t g_grid;
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetLastError(void) { return 0; }
int hipSetDevice(int d) { return d; }
int hipDeviceSynchronize(void) { return 0; }
int hipMemcpy(void* d, const void* s, size_t n, int kind) { return 0; }
int hipMemset(void* d, int v, size_t n) { return 0; }
int hipStreamIsCapturing(void* s, int* status) {
    *status = g_captured_stream && (uintptr_t)s == (uintptr_t)g_captured_stream;
    return 0;
}
int hipThreadExchangeStreamCaptureMode(int* mode) {
    int was = g_mode;
    g_mode = *mode;
    *mode = was;
    return 0;
}
// A capture under way anywhere in the process refuses allocations of a thread
// in the global mode (0) and breaks; a thread in the relaxed mode (2) may allocate.
int hipMalloc(void** p, size_t n) {
    if ((g_captured_stream || g_other_capture) && g_mode != 2) { ++g_refused; return 900; }
    g_last_alloc = g_next; g_last_size = n; g_total += n;
    g_next += (n + 4095) & ~(size_t)4095; ++g_allocs;
    *p = (void*)g_last_alloc;
    return 0;
}
int hipFree(void* p) { g_last_free = (uintptr_t)p; ++g_frees; return 0; }
static dim3_t g_push_grid, g_push_block; static size_t g_push_shmem; static void* g_push_stream;
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t shmem, void* st) {
    g_push_grid = grid; g_push_block = block; g_push_shmem = shmem; g_push_stream = st;
    return 0;
}
int __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, size_t* shmem, void** st) {
    *grid = g_push_grid; *block = g_push_block; *shmem = g_push_shmem; *st = g_push_stream;
    return 0;
}
int hipLaunchKernel(const void* f, dim3_t grid, dim3_t block, void** args, size_t shmem, void* st) {
    g_grid = grid; ++g_launches; return 0;
}
"""

PRELUDE = r"""
import ctypes, sys
S = ctypes.CDLL({stub!r}, mode=ctypes.RTLD_GLOBAL)
L = ctypes.CDLL({lib!r})
vp, u64, u32, i32 = ctypes.c_void_p, ctypes.c_uint64, ctypes.c_uint32, ctypes.c_int
L.gd_apply_sparse.argtypes = [vp, u64, u32, vp, vp, vp, ctypes.c_float, vp]
L.gd_create.argtypes = [ctypes.POINTER(vp), vp, u32]
L.gd_destroy.argtypes = [vp]
def create(offsets):
    "Device bytes that gd_create allocates for a layout, and the allocations it makes."
    h, before, count = vp(), get("g_total", u64), get("g_allocs")
    st = L.gd_create(ctypes.byref(h), (u64 * len(offsets))(*offsets), len(offsets) - 1)
    assert st == 0, st
    L.gd_destroy(h)
    return get("g_total", u64) - before, get("g_allocs") - count
def get(name, t=i32): return t.in_dll(S, name).value
def put(name, v): i32.in_dll(S, name).value = v
def apply(n, clients, nnz, stream=16):
    "Launches of one apply on fake pointers: 2 (bounds and tiles) in the streaming form, 1 in the scattered one."
    ptrs = (vp * clients)(*([4096] * clients))
    before = get("g_launches")
    st = L.gd_apply_sparse(4096, n, clients, ptrs, ptrs, (u64 * clients)(*([nnz] * clients)), 1.0, stream)
    assert st == 0, st
    return get("g_launches") - before
"""


def run(code, tmp_path):
    if not os.path.exists(LIB):
        from paper_1704_05021_amd import build
        build.build()
    src, stub = os.path.join(tmp_path, "stub.c"), os.path.join(tmp_path, "stub.so")
    with open(src, "w") as f:
        f.write(STUB)
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", src, "-o", stub], check=True)
    prog = PRELUDE.format(stub=stub, lib=LIB) + code + "\nprint('STUBBED_OK')\n"
    r = subprocess.run([sys.executable, "-c", prog], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "STUBBED_OK" in r.stdout, f"rc={r.returncode}\n{r.stdout[-2000:]}\n{r.stderr[-4000:]}"
