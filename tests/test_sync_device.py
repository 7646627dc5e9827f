"""fae_sync from a thread whose current device is not the context's: a kernel carries the status word to the host, so
the context's device has to be current at its launch (on the null stream it would run on the other one).
The context's source, compiled for the host against a runtime of a few lines that records launches."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RUNTIME = r"""
#pragma once
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#define __global__
#define __launch_bounds__(...)
struct dim3 { unsigned x, y, z; dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {} };
static dim3 blockIdx, blockDim, threadIdx;
typedef int hipError_t;
typedef void *hipStream_t;
typedef void *hipEvent_t;
enum { hipSuccess = 0, hipHostMallocDefault = 0, hipStreamNonBlocking = 1, hipEventDisableTiming = 2 };
struct hipDeviceProp_t { int multiProcessorCount; };
static int current_device, launches, stray_launches, waits, stray_waits;
static inline const char *hipGetErrorString(int) { return ""; }
static inline int hipGetDeviceCount(int *n) { *n = 2; return 0; }
static inline int hipSetDevice(int d) { current_device = d; return 0; }
static inline int hipGetDeviceProperties(hipDeviceProp_t *p, int) { p->multiProcessorCount = 256; return 0; }
static inline int hipMalloc(void **p, size_t n) { *p = calloc(1, n); return 0; }
static inline int hipHostMalloc(void **p, size_t n, int) { *p = calloc(1, n); return 0; }
static inline int hipHostGetDevicePointer(void **d, void *h, int) { *d = h; return 0; }
static inline int hipFree(void *p) { free(p); return 0; }
static inline int hipHostFree(void *p) { free(p); return 0; }
static inline int hipStreamCreateWithFlags(hipStream_t *s, int) { *s = malloc(1); return 0; }
static inline int hipStreamDestroy(hipStream_t s) { free(s); return 0; }
static inline int hipEventCreate(hipEvent_t *e) { *e = malloc(1); return 0; }
static inline int hipEventCreateWithFlags(hipEvent_t *e, int) { *e = malloc(1); return 0; }
static inline int hipEventDestroy(hipEvent_t e) { free(e); return 0; }
static inline int hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0; return 0; }
static inline int hipGetLastError() { return 0; }
static inline int hipStreamSynchronize(hipStream_t s) { if (!s) { ++waits; stray_waits += current_device != 1; } return 0; }
#define hipLaunchKernelGGL(...) (++launches, stray_launches += current_device != 1)
#define hipExtLaunchKernelGGL(...) (++launches, stray_launches += current_device != 1)
"""

PROGRAM = r"""
#include "fae_ctx.hip"
int32_t fae_bwd_scratch_resolve(fae_ctx *, int, void **out) { *out = nullptr; return 0; }
int main()
{
    fae_ctx *ctx = nullptr;
    if (fae_create(&ctx, 1, nullptr) != FAE_OK)
        return 2;
    (void)hipSetDevice(0);
    launches = stray_launches = waits = stray_waits = 0;
    if (fae_sync(ctx) != FAE_OK || launches < 1 || waits < 1)
        return 3;
    printf("launches %d stray %d, waits %d stray %d\n", launches, stray_launches, waits, stray_waits);
    return stray_launches || stray_waits;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_sync_makes_the_context_s_device_current(tmp_path):
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(RUNTIME)
    (tmp_path / "hip" / "hip_ext.h").write_text("#pragma once\n")
    (tmp_path / "main.cpp").write_text(PROGRAM)
    exe = str(tmp_path / "main")
    subprocess.run(["g++", "-std=c++17", "-w", "-I", str(tmp_path), "-I", os.path.join(ROOT, "paper_2103_00686_amd", "csrc"),
                    "-o", exe, str(tmp_path / "main.cpp")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
