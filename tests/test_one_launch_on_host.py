"""The restore in one launch (lc_decode_one.hip) built for the host: one workgroup of 512 threads as fibers that change places where
lanes exchange values or the workgroup meets, so that the kernel runs from end to end without a GPU.  The blob ends where an
unmapped page begins: reads never leave it, whether it is whole, damaged or refused (include/lc.h).  Against the oracle, bit
for bit."""
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

from oracle import lc_oracle as orc
from tests.test_refused_blob_reads import CLANG, CSRC, SHIM

FIBERS = r"""
#include <ucontext.h>
#include <stdio.h>
// ---- a workgroup's threads as fibers; a thread that waits says for what, and runs on when all that still run of its wavefront
// (or of the workgroup) wait for the same
namespace fibers {
enum { kThreads = 512, kStack = 64 << 10 };
struct Fiber { ucontext_t ctx; char* stack; int state; int waits; unsigned long long value; };      // state: 0 ends, 1 runs; waits: 0 no, 1 wavefront, 2 workgroup
static Fiber f[kThreads];
static ucontext_t home;
static int now;
static unsigned long long seen[kThreads / 64][64], active[kThreads / 64];
static void (*body)();
static void entry() { body(); f[now].state = 0; swapcontext(&f[now].ctx, &home); }
static void wait(int what, unsigned long long v) { f[now].waits = what; f[now].value = v; swapcontext(&f[now].ctx, &home); }
// every lane's value, and which lanes take part
static unsigned long long* exchange(unsigned long long v) { const int w = now / 64; wait(1, v); return seen[w]; }
static void run(void (*b)()) {
    body = b;
    for (int t = 0; t < kThreads; ++t) {
        if (!f[t].stack) f[t].stack = (char*)malloc(kStack);
        getcontext(&f[t].ctx);
        f[t].ctx.uc_stack.ss_sp = f[t].stack; f[t].ctx.uc_stack.ss_size = kStack; f[t].ctx.uc_link = nullptr;
        makecontext(&f[t].ctx, entry, 0);
        f[t].state = 1; f[t].waits = 0;
    }
    for (;;) {
        bool ran = false, left = false;
        for (now = 0; now < kThreads; ++now) {
            if (!f[now].state || f[now].waits) continue;
            threadIdx.x = now; ran = true;
            swapcontext(&home, &f[now].ctx);
        }
        bool all = true;
        for (int w = 0; w < kThreads / 64; ++w) {
            bool together = true, any = false;
            for (int l = 0; l < 64; ++l) { const Fiber& x = f[64 * w + l]; if (x.state) { left = any = true; together = together && x.waits == 1; all = all && x.waits == 2; } }
            if (!any || !together) continue;
            active[w] = 0;
            for (int l = 0; l < 64; ++l) { Fiber& x = f[64 * w + l]; seen[w][l] = x.value; if (x.state) { active[w] |= 1ull << l; x.waits = 0; } }
            ran = true; all = false;
        }
        if (!left) return;
        if (all) { for (auto& x : f) x.waits = 0; ran = true; }
        if (!ran) { puts("threads that wait for different things"); _Exit(4); }
    }
}
}
using fibers::exchange;
static inline int lane() { return fibers::now & 63; }
static inline unsigned long long __ballot(int v) { unsigned long long* x = exchange(v != 0); const unsigned long long a = fibers::active[fibers::now / 64]; unsigned long long m = 0; for (int l = 0; l < 64; ++l) m |= (x[l] && ((a >> l) & 1)) ? 1ull << l : 0; return m; }
static inline int __any(int v) { return __ballot(v) != 0; }
template <typename T> static inline T __shfl(T v, int l, int) { return (T)exchange((unsigned long long)v)[l & 63]; }
template <typename T> static inline T __shfl_xor(T v, int d, int) { return (T)exchange((unsigned long long)v)[lane() ^ d]; }
template <typename T> static inline T __shfl_up(T v, int d, int) { unsigned long long* x = exchange((unsigned long long)v); return (T)x[lane() >= d ? lane() - d : lane()]; }
static inline int read_lane_of(int v, int l) { return (int)exchange((unsigned)v)[l & 63]; }
static inline int dpp(int old, int v, int ctrl, int rows) {
    unsigned long long* x = exchange((unsigned)v);
    const int l = lane(), row = l / 16, shift = ctrl & 15;
    if (!((rows >> row) & 1)) return old;
    if (ctrl == 0x142) return row ? (int)x[16 * row - 1] : old;
    if (ctrl == 0x143) return row >= 2 ? (int)x[31] : old;
    return l % 16 >= shift ? (int)x[l - shift] : old;           // row_shr
}
static inline void __syncthreads() { fibers::wait(2, 0); }
template <typename T, typename U> static inline T atomicMax(T* p, U v) { const T o = *p; if (*p < (T)v) *p = (T)v; return o; }
template <typename T, typename U> static inline T atomicOr(T* p, U v) { const T o = *p; *p |= v; return o; }
#define __builtin_amdgcn_readlane(v, l) read_lane_of((int)(v), (int)(l))
#define __builtin_amdgcn_readfirstlane(v) read_lane_of((int)(v), 0)
#define __builtin_amdgcn_update_dpp(o, v, ctrl, rows, banks, bound) dpp((int)(o), (int)(v), ctrl, rows)
#define __builtin_amdgcn_wave_barrier() ((void)0)
#define __builtin_amdgcn_s_sleep(n) ((void)0)
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_load(p, order, scope) (*(p))
#define __hip_atomic_fetch_add(p, v, order, scope) ((*(p) += (v)) - (v))
template <typename T> static inline bool swap_if(T* p, T* want, T v) { if (*p == *want) { *p = v; return true; } *want = *p; return false; }
#define __hip_atomic_compare_exchange_strong(p, want, v, o1, o2, scope) swap_if((unsigned long long*)(p), (unsigned long long*)(want), (unsigned long long)(v))
#define hipLaunchKernelGGL(kernel, grid, threads, lds, stream, ...) launch([=] { kernel(__VA_ARGS__); })
static std::function<void()> launched;
template <typename F> static void launch(F k) { launched = k; fibers::run([] { launched(); }); }
"""

MAIN = r"""
#include <sys/mman.h>
#include <unistd.h>
using namespace lc;
static unsigned char* load(const char* path, size_t* n) {
    FILE* f = fopen(path, "rb"); fseek(f, 0, SEEK_END); *n = (size_t)ftell(f); rewind(f);
    unsigned char* p = (unsigned char*)malloc(*n + 64); if (fread(p, 1, *n, f) != *n) _Exit(5); fclose(f); return p;
}
// blob, parameters, element type, elements, blobs: what is left of the parameters goes back to the file
int main(int, char** v) {
    size_t nb, nw;
    unsigned char *b = load(v[1], &nb), *w = load(v[2], &nw);
    const size_t page = (size_t)sysconf(_SC_PAGESIZE), room = (nb + page - 1) / page * page;
    unsigned char* m = (unsigned char*)mmap(nullptr, room + page, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    if (m == MAP_FAILED || mprotect(m + room, page, PROT_NONE) != 0) return 2;
    unsigned char* blob = m + room - nb;             // (its size is a multiple of 4, and the kernel asks for no more alignment)
    memcpy(blob, b, nb);
    Workspace* ws = (Workspace*)calloc(1, sizeof(Workspace));
    HostResult* host = (HostResult*)calloc(1, sizeof(HostResult));
    BlobList blobs;
    for (auto& p : blobs.p) p = blob;
    host->bytes[0] = ~0ull;
    uint64_t met[kMeetLines] = {};
    const uint64_t n = strtoull(v[4], 0, 10), epoch = 7;
    gridDim = dim3(1); blockDim = dim3(512); blockIdx = dim3(0);
    blockIdx.x = 0;
    launch_decode_one(blobs, atoi(v[5]), w, n, atoi(v[3]), ~0ull, ws, epoch, host, met, 4, nullptr);
    const int status = (host->dec_status >> 8) == epoch ? (int)(host->dec_status & 255) : host->bytes[0] == ~0ull ? 99 : 0;
    FILE* f = fopen(v[2], "wb"); fwrite(w, 1, nw, f); fclose(f);
    printf("status %d\n", status);
    return 0;
}
"""

TYPES = {"fp32": (0, np.float32), "bf16": (1, np.uint16), "fp16": (2, np.float16), "fp64": (3, np.float64)}


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not os.path.exists(CLANG) or shutil.which("hipcc") is None:
        pytest.skip("needs the ROCm compiler")
    d = tmp_path_factory.mktemp("one")
    (d / "hip").mkdir()
    shim = SHIM[:SHIM.index("// what lanes exchange")] + "static inline unsigned __builtin_alignbit(unsigned a, unsigned b, unsigned s) { return (unsigned)((((unsigned long long)a << 32) | b) >> (s & 31)); }\n"
    (d / "hip" / "hip_runtime.h").write_text(shim + FIBERS)
    for name in ("lc_device.h", "lc_internal.h", "lc_meeting.h", "lc_decode_one.hip"):
        text = open(os.path.join(CSRC, name)).read()
        text = re.sub(r"\basm( volatile)?\([^;]*\);", ";", text)
        text = text.replace("__builtin_amdgcn_alignbit", "__builtin_alignbit")
        (d / name).write_text(text)
    (d / "main.cpp").write_text('#include <initializer_list>\n#include <type_traits>\n#include <functional>\n#include "lc_decode_one.hip"\n' + MAIN)
    res = subprocess.run([CLANG, "-x", "c++", "-std=c++17", "-O1", "-ffp-contract=off", "-w", "-I", str(d), str(d / "main.cpp"), "-o", str(d / "one")], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]
    return d


def encoded(name, n, nbits, kind, seed):
    rng = np.random.RandomState(seed)
    if kind == "few":
        e = np.zeros(n); e[:n // 2] = np.floor(3 * rng.rand(n // 2)); e[n // 2 + rng.randint(0, n - n // 2, 20)] = 2
    elif kind == "quiet":
        e = np.zeros(n)
    else:
        e = np.floor(-np.log2(np.maximum(rng.rand(n), 2.0 ** -15)))
        e = np.where(e < 15, 15 - e, 0)                                   # "deep": long codes among short ones
    d = np.where(e > 0, np.exp2(e - 9) * (1 + 0.5 * rng.rand(n)), 0)
    if name == "fp64":
        return orc.encode64(d, np.zeros(n), nbits)
    if name == "bf16":
        return orc.encode_t((d.astype(np.float32).view(np.uint32) >> 16).astype(np.uint16), np.zeros(n, np.uint16), nbits, orc.DT_BF16)
    if name == "fp16":
        return orc.encode_t(d.astype(np.float16), np.zeros(n, np.float16), nbits, orc.DT_F16)
    return orc.encode(d.astype(np.float32), np.zeros(n, np.float32), nbits)


def oracle(name, blob, x):
    if name == "fp64":
        orc.decode64(blob, x)
    elif name == "fp32":
        orc.decode(blob, x)
    else:
        orc.decode_t(blob, x, orc.DT_BF16 if name == "bf16" else orc.DT_F16)


def run(program, name, blob, x, count=1, n=None):
    blob.tofile(str(program / "blob")); x.tofile(str(program / "x"))
    res = subprocess.run([str(program / "one"), str(program / "blob"), str(program / "x"), str(TYPES[name][0]), str(x.size if n is None else n), str(count)],
                         capture_output=True, text=True, timeout=100)
    assert res.returncode == 0, (res.returncode, res.stdout[-500:])      # (-11: a read behind the blob's end)
    return int(res.stdout.split()[-1]), np.fromfile(str(program / "x"), x.dtype)


def parameters(name, n, seed):
    x = np.random.RandomState(seed).randn(n)
    return (x.astype(np.float32).view(np.uint32) >> 16).astype(np.uint16) if name == "bf16" else x.astype(TYPES[name][1])


@pytest.mark.parametrize("name", list(TYPES))
@pytest.mark.parametrize("n,kind,nbits", [(16384, "deep", 4), (16384, "deep", 3), (5003, "deep", 4), (16384, "few", 2), (16383, "few", 2), (16384, "quiet", 3), (7, "deep", 1)])
def test_as_the_oracle(program, name, n, kind, nbits):
    blob, x = encoded(name, n, nbits, kind, n), parameters(name, n, 3)
    for count in (1, 3):
        want = x.copy()
        for _ in range(count):
            oracle(name, blob, want)
        status, got = run(program, name, blob, x, count)
        assert status == 0 and np.array_equal(got.view(np.uint8), want.view(np.uint8)), count


@pytest.mark.parametrize("kind", ["deep", "few", "quiet"])
def test_damaged_and_refused(program, kind):
    """Header, offsets, lane lengths, strings: the oracle's verdict, nothing touched on a refusal, nothing read behind the blob."""
    n, name = 3000, "fp32"
    blob, x = encoded(name, n, 3, kind, 1), parameters(name, n, 5)
    rng = np.random.RandomState(2)
    bits = [8 * 8, 8 * 41, 8 * 66 + 1, 8 * 512, 8 * 516, 8 * 516 + 31] + list(rng.randint(8 * 528, 8 * (528 + 128), 6)) + list(rng.randint(8 * (528 + 128), 8 * blob.size, 6))
    for at in bits:
        bad = blob.copy(); bad[at // 8] ^= 1 << (at % 8)
        want, verdict = x.copy(), 0
        try:
            oracle(name, bad, want)
        except orc.OracleError as e:
            want, verdict = x, e.status
        status, got = run(program, name, bad, x)
        assert status == verdict and (verdict or np.array_equal(got.view(np.uint8), want.view(np.uint8))), (at, status, verdict)
        if verdict:
            assert np.array_equal(got.view(np.uint8), x.view(np.uint8)), at      # (a single chunk is restored wholly or not at all)
    # a header alone, refused for what it says: n, the element type, a delta that was not finite
    head = blob[:512].copy(); head[8] ^= 1
    assert run(program, name, head, x)[0] == 1
    head = blob[:512].copy(); head[60] = 1
    assert run(program, name, head, x)[0] == 1
    w = np.full(n, np.inf, np.float32)
    try:
        orc.encode(w, np.zeros(n, np.float32), 3)
        raise AssertionError("finite?")
    except orc.OracleError as e:
        assert run(program, name, np.frombuffer(bytes(e.header), np.uint8).copy(), x)[0] == 4
