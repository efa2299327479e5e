"""What the restoring kernels read of a blob that the check has refused: nothing (include/lc.h: reads never leave the blob, and
the blob handed in may be shorter than the caller's n asks for).  The kernels' own source is built for the host, with a few
stand-ins for the device's types and built-ins, and every thread of some workgroups is run, one after the other, on a blob that
ends where an unmapped page begins."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2009_13003_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"

SHIM = r"""
#pragma once
#include <stdint.h>
#include <stddef.h>
#include <stdlib.h>
#include <math.h>
#include <string.h>
#define __device__
#define __host__
#define __global__ static
#define __shared__ static
#define __forceinline__ inline
#define __noinline__
#define __launch_bounds__(...)
struct dim3 { unsigned x, y, z; dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {} };
static dim3 threadIdx, blockIdx, blockDim, gridDim;
typedef void* hipStream_t;
struct float4 { float x, y, z, w; };
struct uint4 { unsigned x, y, z, w; };
struct uint2 { unsigned x, y; };
struct double2 { double x, y; };
static inline float4 make_float4(float a, float b, float c, float d) { return {a, b, c, d}; }
static inline uint4 make_uint4(unsigned a, unsigned b, unsigned c, unsigned d) { return {a, b, c, d}; }
static inline uint2 make_uint2(unsigned a, unsigned b) { return {a, b}; }
static inline double2 make_double2(double a, double b) { return {a, b}; }
template <typename T, typename U> static inline T pun(U u) { T t; memcpy(&t, &u, sizeof t); return t; }
static inline unsigned __float_as_uint(float f) { return pun<unsigned>(f); }
static inline int __float_as_int(float f) { return pun<int>(f); }
static inline float __uint_as_float(unsigned u) { return pun<float>(u); }
static inline long long __double_as_longlong(double d) { return pun<long long>(d); }
static inline double __hiloint2double(int hi, int lo) { return pun<double>(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo); }
static inline float __fadd_rn(float a, float b) { return a + b; }
static inline float __fsub_rn(float a, float b) { return a - b; }
static inline double __dadd_rn(double a, double b) { return a + b; }
static inline double __dsub_rn(double a, double b) { return a - b; }
template <typename T> static inline T min(T a, T b) { return a < b ? a : b; }
template <typename T> static inline T max(T a, T b) { return a < b ? b : a; }
static inline unsigned __lane_id() { return threadIdx.x & 63; }
static inline int __popc(unsigned v) { return __builtin_popcount(v); }
static inline int __popcll(unsigned long long v) { return __builtin_popcountll(v); }
// what lanes exchange, and what a refused call must not come to
template <typename T> static inline T stop(T v) { _Exit(3); return v; }
static inline unsigned long long __ballot(int v) { return stop((unsigned long long)v); }
static inline int __any(int v) { return stop(v); }
template <typename T> static inline T __shfl_xor(T v, int, int) { return stop(v); }
template <typename T> static inline T __shfl(T v, int, int) { return stop(v); }
template <typename T> static inline T atomicMax(T*, T v) { return stop(v); }
static inline void __syncthreads() { _Exit(3); }
#define __builtin_amdgcn_readlane(v, l) stop((int)(v))
#define __builtin_amdgcn_update_dpp(o, v, a, b, c, d) stop((int)(v))
#define __builtin_amdgcn_alignbit(a, b, s) stop((unsigned)(a))
#define __builtin_amdgcn_wave_barrier() ((void)0)
#define __builtin_amdgcn_readfirstlane(v) (v)
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_load(p, order, scope) (*(p))
#define hipLaunchKernelGGL(...) ((void)0)
"""

MAIN = r"""
#include <sys/mman.h>
#include <unistd.h>
#include <stdio.h>
using namespace lc;
template <typename F> static void every_thread(unsigned blocks, unsigned threads, F f) {
    gridDim = dim3(blocks); blockDim = dim3(threads);
    for (unsigned b : {0u, 1u, blocks - 1})
        for (unsigned t = 0; t < threads; ++t) { blockIdx.x = b; threadIdx.x = t; f(); }
}
int main() {
    const size_t page = (size_t)sysconf(_SC_PAGESIZE);
    char* m = (char*)mmap(nullptr, 3 * page, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    if (m == MAP_FAILED || mprotect(m + 2 * page, page, PROT_NONE) != 0) return 2;
    const uint8_t* blob = (const uint8_t*)m + 2 * page - LEFT;      // LEFT bytes of it, then nothing
    Workspace* ws = (Workspace*)calloc(1, sizeof(Workspace));
    HostResult* host = (HostResult*)calloc(1, sizeof(HostResult));
    const uint64_t n = 1ull << 28, epoch = 7;
    const unsigned nchunks = (unsigned)num_chunks_of(n);
    float* w_ref = nullptr;
    ws->dec_status = (epoch << 8) | 4u;
    memset(ws->dec_set, PATTERN, sizeof ws->dec_set);               // what an earlier call, or nobody, left in the tables
    every_thread(2304, 256, [&] { k_decode<kF32>(blob, w_ref, n, ws, nchunks, 1, epoch, host, 2048, 0); });
    every_thread(2304, 256, [&] { k_decode<kBF16>(blob, w_ref, n, ws, nchunks, 1, epoch, host, 2048, 0); });
    every_thread(2304, 256, [&] { k_decode<kF16>(blob, w_ref, n, ws, nchunks, 1, epoch, host, 2048, 0); });
    every_thread(2304, 256, [&] { k_decode<kF64>(blob, w_ref, n, ws, nchunks, 1, epoch, host, 2048, 0); });
    every_thread(2304, 256, [&] { k_decode<kF32, true>(blob, w_ref, n, ws, nchunks, 1, epoch, host, 2048, 0); });
    BlobList blobs;
    for (int i = 0; i < kMaxSets; ++i) blobs.p[i] = blob;
    every_thread(2048, 64, [&] { k_decode_fused<4, false, kF32>(blobs, 0u, w_ref, n, ws, nchunks, epoch, host, 4096u); });
    every_thread(2048, 64, [&] { k_decode_fused<4, true, kBF16>(blobs, 0u, w_ref, n, ws, nchunks, epoch, host, 4096u); });
    puts("nothing read");
    return 0;
}
"""


@pytest.mark.skipif(not os.path.exists(CLANG) or shutil.which("hipcc") is None, reason="needs the ROCm compiler")
def test_a_refused_blob_is_not_read_by_the_sweeps(tmp_path):
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(SHIM)
    for name in ("lc_device.h", "lc_internal.h", "lc_decode.hip"):
        text = open(os.path.join(CSRC, name)).read()
        text = re.sub(r"extern __shared__ (\w+) (\w+)\[\];", r"static \1 \2[1];", text)
        text = re.sub(r"\basm( volatile)?\([^;]*\);", ";", text)           # (empty statements that only pin registers)
        (tmp_path / name).write_text(text)
    (tmp_path / "main.cpp").write_text('#include <initializer_list>\n#include <type_traits>\n#include "lc_decode.hip"\n' + MAIN)
    for left, pattern in ((512, 0), (512, 0xFF), (16, 0x55)):              # a header alone (a delta that is not finite), and less
        exe = tmp_path / ("refused_%d_%d" % (left, pattern))
        res = subprocess.run([CLANG, "-x", "c++", "-std=c++17", "-O0", "-w", "-I", str(tmp_path), "-DLEFT=%d" % left, "-DPATTERN=%d" % pattern,
                              str(tmp_path / "main.cpp"), "-o", str(exe)], capture_output=True, text=True)
        assert res.returncode == 0, res.stderr[-3000:]
        run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
        assert run.returncode == 0 and "nothing read" in run.stdout, (left, pattern, run.returncode)
