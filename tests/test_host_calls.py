"""The host side of the library (lc_api.hip) built for the CPU, with a stand-in for the HIP runtime and for the kernels' launchers
that notes what is launched: the order of launches where calls in one launch are given up, and what another thread's call does that
takes the same scratch area before the first one's outcome is known (made to come in while the first thread waits, the lock
dropped); what is learned from a call that was given up; and which way lists of blobs go."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2009_13003_amd", "csrc")

HIP = r"""
#pragma once
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
#define __device__
#define __host__
#define __align__(x)
typedef int hipError_t;
typedef void* hipStream_t;
typedef struct FakeEvent { hipStream_t s; }* hipEvent_t;
enum { hipSuccess = 0, hipErrorUnknown = 999 };
enum { hipDeviceAttributeMultiprocessorCount, hipHostMallocMapped = 1, hipHostMallocPortable = 2, hipEventDisableTiming = 2 };
hipError_t hipStreamSynchronize(hipStream_t s);
hipError_t hipGetLastError();
static inline hipError_t hipGetDevice(int* d) { *d = 0; return 0; }
static inline hipError_t hipSetDevice(int) { return 0; }
static inline hipError_t hipDeviceGetAttribute(int* v, int, int) { *v = 256; return 0; }
static inline hipError_t hipDeviceSynchronize() { return 0; }
static inline hipError_t hipMalloc(void** p, size_t n) { *p = aligned_alloc(256, (n + 255) / 256 * 256); return *p ? 0 : 1; }
static inline hipError_t hipFree(void* p) { free(p); return 0; }
static inline hipError_t hipHostMalloc(void** p, size_t n, int) { *p = calloc(1, n); return 0; }
static inline hipError_t hipHostFree(void* p) { free(p); return 0; }
static inline hipError_t hipHostGetDevicePointer(void** p, void* h, int) { *p = h; return 0; }
static inline hipError_t hipMemset(void* p, int v, size_t n) { memset(p, v, n); return 0; }
static inline hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t) { memset(p, v, n); return 0; }
static inline hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)calloc(1, sizeof(FakeEvent)); return 0; }
static inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, int) { return hipEventCreate(e); }
static inline hipError_t hipEventDestroy(hipEvent_t e) { free(e); return 0; }
static inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { e->s = s; return 0; }
static inline hipError_t hipEventQuery(hipEvent_t) { return 0; }            // every stream is through with its work at once
static inline hipError_t hipEventSynchronize(hipEvent_t) { return 0; }
static inline hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0; return 0; }
static inline hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t) { return 0; }
static inline hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, int) { return 0; }
#define HIP_SYMBOL(x) (x)
static inline hipError_t hipGetSymbolAddress(void** p, void* x) { *p = x; return 0; }
"""

MAIN = r"""
#include "lc_api.hip"
#include <functional>
#include <stdio.h>
#include <string>

// ---- what is launched: a letter each, and what the stand-ins leave for the host
//   0 k_reset   r k_reset_one   E / D one launch   h first sweep   t table   s single sweep   p second sweep   P placement
//   c check     v verify        d restore          f / g fused restore, by symbols or by pairs of them
static std::string launched;
static bool meet = true;                 // whether the workgroups of a call in one launch meet
static uint64_t blob_bytes = 1000;       // of every blob that is checked or restored, and its longest code
static uint32_t blob_max_len = 3, blob_kept = 3;
static std::vector<uint32_t> kept_of;    // ... of each blob of a list, where they differ
static std::vector<uint64_t> bytes_of;
static int fused_fits = 8;               // blobs that a fused sweep by symbols takes at once
static int fail_launches = 0;            // the next launches that fail
static std::function<void()> waiting;    // runs (once) in a thread that waits for its stream
hipError_t hipGetLastError() { if (fail_launches > 0) { --fail_launches; return hipErrorUnknown; } return 0; }
hipError_t hipStreamSynchronize(hipStream_t) { if (waiting) { auto f = waiting; waiting = nullptr; f(); } return 0; }

namespace lc {
static void done(Result* r) { r->bytes = 1000; r->status = 0; r->used_cache = 0; r->listed = 0; }
void launch_reset(Workspace*, uint32_t*, uint32_t*, hipStream_t) { launched += '0'; }
void launch_reset_chunks(Workspace*, uint32_t*, uint32_t*, uint32_t, hipStream_t) {}
void launch_reset_one(Workspace*, hipStream_t) { launched += 'r'; }
void launch_hist(const void*, const void*, uint64_t, int, Workspace*, uint32_t*, uint8_t*, KeyPlanes, const Tuning&, hipStream_t) { launched += 'h'; }
void launch_pack_keys(const void*, const void*, uint64_t, Workspace*, uint32_t*, uint32_t*, const uint32_t*, const uint32_t*, KeyPlanes, uint32_t*, uint32_t, hipStream_t) { launched += 'p'; }
void launch_table(Workspace*, uint64_t, int, int, uint32_t*, const uint32_t*, uint32_t*, hipStream_t) { launched += 't'; }
void launch_spec_table(Workspace*, const TableCache*, uint64_t, int, int, uint32_t*, hipStream_t) {}
void launch_spec_sweep(const void*, const void*, uint64_t, int, Workspace*, uint32_t*, uint32_t*, uint32_t*, uint32_t, const Tuning&, hipStream_t) { launched += 's'; }
void launch_pack(const void*, const void*, uint64_t, int, Workspace*, uint32_t*, uint32_t*, const uint32_t*, const uint32_t*, const uint8_t*, uint32_t*, uint32_t, const Tuning&, hipStream_t) { launched += 'p'; }
bool pack_needs_list(uint64_t, int, const Tuning&) { return false; }
void launch_place(uint8_t*, Workspace*, const uint32_t*, const uint32_t*, const uint32_t*, uint32_t, uint64_t, uint32_t*, Result* r, TableCache*, int, int, bool, hipStream_t) { launched += 'P'; done(r); }
void launch_encode_one(const void*, const void*, uint64_t, int, int, uint8_t*, Workspace*, uint32_t*, TableCache*, Result* r, uint64_t (&)[kMeetLines], int, hipStream_t) { launched += 'E'; if (meet) done(r); }
void launch_batch_encode(const BatchArgs&, const Tuning&, hipStream_t) {}
void launch_batch_decode(const BatchDecArgs&, const Tuning&, hipStream_t) {}
void launch_dec_check(const BlobList&, int, int count, uint64_t, int, uint64_t, Workspace*, uint64_t, HostResult* host, hipStream_t) {
    launched += 'c';
    for (int i = 0; i < count; ++i) { host->bytes[i] = bytes_of.empty() ? blob_bytes : bytes_of[i]; host->max_len[i] = blob_max_len; host->kept[i] = kept_of.empty() ? blob_kept : kept_of[i]; }
}
void launch_decode(const uint8_t*, void* w_ref, uint64_t, int, Workspace*, int, uint64_t, HostResult*, const Tuning&, hipStream_t) { launched += w_ref ? 'd' : 'v'; }
void launch_decode_one(const BlobList&, int count, void*, uint64_t, int, uint64_t, Workspace*, uint64_t, HostResult* host, uint64_t (&)[kMeetLines], int, hipStream_t) {
    launched += 'D';
    if (meet) for (int i = 0; i < count; ++i) host->bytes[i] = blob_bytes;
}
void launch_decode_fused(const BlobList&, int, int, void*, uint64_t, int, Workspace*, uint64_t, HostResult*, uint32_t, bool, const Tuning&, hipStream_t) { launched += 'f'; }
void launch_decode_pairs(const BlobList&, int, int, void*, uint64_t, int, Workspace*, uint64_t, HostResult*, double, bool, const Tuning&, hipStream_t) { launched += 'g'; }
size_t fused_lds_bytes(int count, uint32_t) { return count <= fused_fits ? 1 : 1 << 20; }
}  // namespace lc

static int wrong = 0;
static void expect(const char* what, const std::string& want) {
    if (launched != want) { printf("%s: %s, not %s\n", what, launched.c_str(), want.c_str()); ++wrong; }
    launched.clear();
}
alignas(256) static char mem[4][256];
static const uint64_t kShort = 40 * 16384, kShortest = 3 * 16384, kLong = 600 * 16384;
static void* stream(intptr_t i) { return (void*)i; }
static lc_ssize encode(uint64_t n, intptr_t s) { return lc_encode((const float*)mem[0], (const float*)mem[1], n, 3, mem[2], stream(s)); }
static int encode_async(uint64_t n, intptr_t s) { return lc_encode_async((const float*)mem[0], (const float*)mem[1], n, 3, mem[2], nullptr, stream(s)); }
static lc_ssize decode(uint64_t n, intptr_t s) { return lc_decode(mem[2], (float*)mem[0], n, stream(s)); }
static lc_ssize decode_many(int count, uint64_t n, intptr_t s) {
    const void* blobs[LC_MAX_MANY];
    for (auto& b : blobs) b = mem[2];
    return lc_decode_many(blobs, count, (float*)mem[0], n, stream(s));
}
static lc_ssize decode_many_t(int count, uint64_t n, int dtype, int offset = 0) {
    const void* blobs[LC_MAX_MANY];
    for (auto& b : blobs) b = mem[2];
    return lc_decode_many_t(blobs, count, mem[0] + offset, n, dtype, stream(1));
}
static void ok(lc_ssize r, lc_ssize want = 1000) { if (r != want) { printf("result %lld, not %lld\n", (long long)r, (long long)want); ++wrong; } }
static std::string times(int k, const char* x) { std::string r; while (k--) r += x; return r; }
static void fresh() { lc_shutdown(); meet = true; waiting = nullptr; launched.clear(); }
// the one scratch area of a caller: every stream's calls take it
static void* caller_area() {
    const size_t bytes = (lc_workspace_bytes(kLong, 3) + 255) / 256 * 256;
    void* p = aligned_alloc(256, bytes);
    lc_set_workspace(p, bytes);
    return p;
}

SCENARIOS
int main() { scenarios(); lc_shutdown(); if (!wrong) puts("as expected"); return wrong != 0; }
"""

# each: the body of scenarios()
GIVEN_UP = r"""
static void scenarios() {
    // alone
    fresh(); ok(encode(kShort, 1)); expect("fresh area", "0E");
    ok(encode(kShort, 1)); ok(encode(kLong, 1)); ok(encode(kShort, 1)); expect("a larger area, then nothing to clear", "E0htpPE");
    meet = false; ok(encode(kShort, 1)); expect("given up", "ErhtpP");
    meet = true; ok(encode(kLong, 1)); expect("and cleared", "htpP");

    for (int user = 0; user < 2; ++user)
        for (int second = 1; second <= 2; ++second)                     // the second call's stream (the area of another one counts as idle)
            for (int kind = 0; kind < 4; ++kind) {
                fresh();
                void* area = user ? caller_area() : nullptr;
                ok(encode(kShort, 1)); ok(encode(kLong, 1)); launched.clear();
                // another thread's call comes in while the first one's outcome is open
                int ticket = -1;
                meet = false;
                waiting = [&] {
                    meet = true;
                    if (kind == 0) ticket = encode_async(kLong, second);
                    if (kind == 1) ok(encode(kLong, second));
                    if (kind == 2) ticket = encode_async(kShortest, second);
                    if (kind == 3) ok(encode(kShortest, second));            // fewer counters to look at than the first
                };
                ok(encode(kShort, 1));
                if (ticket >= 0) ok(lc_encode_wait(ticket, nullptr));
                expect("behind an open call", std::string(kind == 3 ? "ErE" : "ErhtpP") + "rhtpP");
                // and one behind a call that did meet, while a third is open
                waiting = [&] { waiting = [&] { ok(encode(kLong, second)); }; ok(encode(kShort, second)); };
                ok(encode(kShort, 1));
                expect("two open calls", "ErErhtpP");
                ok(encode(kLong, second)); expect("none open", "htpP");
                fresh();
                free(area);
            }

    fresh(); ok(encode(kShort, 1)); launched.clear();
    fail_launches = 1; ok(encode(kShort, 1), -LC_ERR_HIP); ok(encode(kLong, 1)); expect("a launch that failed", "E0htpP");
    // 2-byte types up to 448 chunks where they are aligned and have no cache
    fresh();
    for (int dtype : {LC_F32, LC_BF16, LC_F16})
        for (int offset : {0, 2, 4, 8})
            for (int cached = 0; cached < 2; ++cached)
                for (uint64_t chunks : {448, 449, 512, 513}) {
                    if (dtype == LC_F32 && offset == 2) continue;
                    const char* w = mem[0] + offset;
                    const bool one = chunks <= (dtype == LC_F32 || cached || offset % 8 ? 512u : 448u);
                    ok(cached ? lc_encode_cached_t(w, mem[1], chunks * 16384, 3, mem[2], dtype, mem[3], nullptr, stream(1))
                              : lc_encode_t(w, mem[1], chunks * 16384, 3, mem[2], dtype, stream(1)));
                    if (launched[0] == '0') launched.erase(0, 1);           // (the area grows)
                    expect("by size", one ? "E" : cached ? "stpP" : "htpP");
                }
    // restores: the counters are known again after a refusal, a given-up call, a launch that failed
    fresh(); ok(decode(kShort, 1)); expect("fresh area", "D");
    meet = false; ok(decode(kShort, 1)); meet = true; ok(decode(kShort, 1)); expect("given up", "DcdrD");
    fail_launches = 1; ok(decode(kShort, 1), -LC_ERR_HIP); ok(decode(kShort, 1)); expect("a launch that failed", "DrD");
    ok(encode(kLong, 1)); expect("an area that only restores used", "0htpP");
}
"""

REST = r"""
static void scenarios() {
    // the calls behind one that was given up do not try: 16, then twice as many each time, up to 1024, until one is not given up
    for (int what = 0; what < 3; ++what) {
        fresh();
        const char* one = what == 0 ? "E" : "D", *several = what == 0 ? "htpP" : what == 1 ? "cd" : "cf";
        auto call = [&] { ok(what == 0 ? encode(kShort, 1) : what == 1 ? decode(kShort, 1) : decode_many(2, kShort, 1), what == 2 ? 2000 : 1000); };
        call(); launched.clear();
        for (int round = 0; round < 2; ++round) {
            for (int len = 16; len <= 4096; len *= 2) {
                const int rest = len < 1024 ? len : 1024;
                meet = false; call(); meet = true;
                // (what the last one left on the counters is cleared by the next that needs them, or adds to the counts)
                expect("given up", std::string(len > 16 && what ? "r" : "") + one + (what == 0 ? "r" : "") + several);
                for (int i = 0; i < rest; ++i) call();
                expect("resting", times(rest, several));
            }
            call(); expect("tried again", std::string(what ? "r" : "") + one);
            for (int i = 0; i < 5; ++i) call();
            expect("and met", times(5, one));
        }
    }
    // a restore of several blobs in one launch waits with the lock dropped: other calls go on
    fresh(); ok(decode(kShort, 1)); launched.clear();
    waiting = [] { ok(encode(kLong, 2)); };
    ok(decode_many(2, kShort, 1), 2000); expect("beside a restore of several blobs", "D0htpP");
    meet = false; waiting = [] { ok(encode(kLong, 2)); };
    ok(decode_many(2, kShort, 1), 2000); expect("... that is given up", "DhtpPcf");
}
"""

MANY = r"""
static void scenarios() {
    // several blobs: in one launch as they come where that is the faster way whatever they hold, else by what the check finds
    fresh();
    const uint64_t small = 64 * 16384, large = 300 * 16384, beyond = 513 * 16384;
    auto is = [&](const char* want, int count, uint64_t n, int dtype, int offset = 0) {
        const std::string what = std::to_string(count) + " blobs, " + std::to_string(n / 16384) + " chunks, type " + std::to_string(dtype);
        ok(decode_many_t(count, n, dtype, offset), (lc_ssize)blob_bytes * count);
        expect(what.c_str(), want);
    };
    for (int dtype : {LC_F32, LC_BF16, LC_F16}) {
        for (uint32_t len : {7u, 8u}) {
            blob_max_len = len;
            is("D", 1, small, dtype); is("D", 5, small, dtype); is(len > 7 ? "cD" : "cf", 6, small, dtype);
            is("D", 3, large, dtype); is(len > 7 ? "cD" : "cf", 4, large, dtype);
            is("D", 64, small, dtype, dtype == LC_F32 ? 4 : 2); is("D", 8, large, dtype, dtype == LC_F32 ? 8 : 4);
            is("cf", 2, beyond, dtype);
        }
    }
    blob_max_len = 3;
    blob_bytes = 16384;
    is("D", 8, small, LC_F64); is("cdd", 2, large, LC_F64); is("cdd", 2, beyond, LC_F64);
    blob_bytes = large / 4;
    is("cD", 2, large, LC_F64); is("cD", 8, large, LC_F64, 8); is("cdd", 2, beyond, LC_F64);
    // which of the two kernels takes a list, and in how many sweeps: of few symbols the second from 5 blobs and 3 or 6 chunks per
    // compute unit on, or where the first takes less than 4 at a time, of 16 from 3 blobs on; either shares them out evenly
    blob_bytes = 1000;
    for (uint64_t per_cu : {2, 3, 5, 6, 20})
        for (int fits : {2, 3, 4, 6, 8})
            for (int count = 2; count <= 20; ++count) {
                const int in_fused = (count + fits - 1) / fits;
                const uint64_t size = (per_cu * 256 + 1) * 16384;
                fused_fits = fits;
                for (uint32_t kept : {0u, 7u}) {
                    blob_kept = kept;
                    std::string want = "c";
                    for (int left = count; left > 0;) {              // (the last few of 9, 10, ... may be too few for the second)
                        const int sweeps = (left + 7) / 8, pairs = (left + sweeps - 1) / sweeps, rounds = (left + fits - 1) / fits;
                        const bool second = pairs >= 5 && (per_cu >= 6 || (per_cu >= 3 ? fits != 4 || left % fits : fits < 4));
                        want += second ? "g" : "f";
                        left -= second ? pairs : (left + rounds - 1) / rounds;
                    }
                    is(want.c_str(), count, size, LC_F32);
                    is(("c" + times((count + 7) / 8, "g")).c_str(), count, size, LC_BF16, 2);
                }
                if (fits == 3) continue;
                blob_kept = 15;
                const int sweeps = (count + 3) / 4;
                if (count > 2 && count != 5) is(("c" + times(sweeps < in_fused ? sweeps : in_fused, sweeps < in_fused ? "g" : "f")).c_str(), count, size, LC_F16);
                blob_max_len = 8;
                if (count > 2 && count != 5) is(("c" + times(sweeps, "g")).c_str(), count, size, LC_F32);
                blob_max_len = 3;
            }
    // lists of both kinds: one blob of more than 8 symbols takes its neighbours along, but for a run that has sweeps of its own
    auto mixed = [&](const char* want, std::vector<uint32_t> kept, uint64_t chunks, int offset = 0) {
        kept_of = kept;
        is(want, (int)kept.size(), chunks * 16384, LC_F32, offset);
        kept_of.clear();
    };
    std::vector<uint32_t> turns;
    for (int i = 0; i < 7; ++i) { turns.push_back(7); turns.push_back(15); }
    for (uint64_t chunks : {600, 8192}) {
        for (int offset : {0, 4}) {
            fused_fits = 3; mixed(offset ? "cgggg" : "cggff", turns, chunks, offset);
            fused_fits = 2; mixed("cgggg", turns, chunks, offset);
            mixed("cg", {0, 15, 0, 15}, chunks, offset); mixed("cgg", {15, 15, 15, 0, 15, 15, 15}, chunks, offset);
        }
        fused_fits = 8; mixed("cff", turns, chunks); mixed("cgggg", turns, chunks, 8);
        fused_fits = 4; blob_max_len = 8; mixed("cgggg", turns, chunks); blob_max_len = 3;
    }
    mixed("cfg", {15, 7, 7, 7, 7, 7, 7}, 8192); mixed("cgf", {7, 7, 7, 7, 7, 7, 15}, 8192); blob_max_len = 8; mixed("cfg", {7, 7, 7, 7, 15, 15, 15}, 8192); blob_max_len = 3;
    mixed("cdg", {15, 7, 7, 7, 7, 7, 7}, 8192, 4); mixed("cgd", {7, 7, 7, 7, 7, 7, 15}, 600, 4); mixed("cdggd", {15, 7, 7, 7, 7, 7, 7, 7, 7, 7, 7, 15}, 8192, 4);
    // ... and sparse blobs (532 words a chunk here) do not go with dense ones (564) of the other kind, where some codes are long
    blob_max_len = 8;
    const uint64_t chunks = 8192, sparse = 512 + 4 * (chunks + 4) + 4 * 532 * chunks, more = sparse + 4 * 32 * chunks;
    auto kinds = [&](const char* want, std::vector<uint32_t> kept, std::vector<uint64_t> bytes, int offset = 0) {
        kept_of = kept; bytes_of = bytes;
        uint64_t total = 0;
        for (uint64_t b : bytes) total += b;
        ok(decode_many_t((int)kept.size(), chunks * 16384, LC_F32, offset), (lc_ssize)total);
        expect(want, want);
        kept_of.clear(); bytes_of.clear();
    };
    kinds("cfff", {15, 0, 15}, {more, sparse, more}); kinds("cddd", {15, 0, 15}, {more, sparse, more}, 4);
    kinds("cg", {15, 7, 15}, {more, more, more}); kinds("cg", {15, 0, 15}, {sparse, sparse, sparse}); kinds("cfg", {0, 15, 15, 15}, {sparse, more, more, sparse});
    kinds("cgf", {7, 7, 15, 7}, {more, sparse, more, sparse});
    blob_max_len = 3; kinds("cf", {15, 0, 15}, {more, sparse, more});
    // few chunks: the second where the first takes less than 4 dense ones, and of 2-byte elements 7 or 8 sparse ones
    blob_bytes = 1000; blob_kept = 7;
    for (int fits : {3, 4, 6}) {
        fused_fits = fits;
        is(fits == 3 ? "cg" : "cff", 8, small, LC_F32); is(fits == 4 ? "cff" : "cg", 8, small, LC_BF16); is(fits == 3 ? "cgg" : fits == 4 ? "cfff" : "cff", 12, small, LC_F16);
        is(fits == 3 ? "cfg" : fits == 4 ? "cfff" : "cff", 10, small, LC_F32);
    }
    fused_fits = 8;
    is("cd", 1, beyond, LC_F32, 4); is("cd", 1, beyond, LC_BF16, 2); is("cf", 1, beyond, LC_F32);
    blob_kept = 3; fused_fits = 8;
    // given up behind the check
    blob_bytes = 1000; blob_max_len = 9; meet = false;
    is("cDcff", 16, small, LC_F32);
    meet = true;
    is("cff", 16, small, LC_F32);
    // the check of the strings comes first where that is asked for
    fresh();
    lc_set_option(LC_OPT_VERIFY_FIRST, 1);
    is("cvvf", 2, small, LC_F32);
    lc_set_option(LC_OPT_VERIFY_FIRST, 0);
    is("D", 2, small, LC_F32);
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
@pytest.mark.parametrize("scenarios", ["GIVEN_UP", "REST", "MANY"])
def test_order_of_launches(tmp_path, scenarios):
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(HIP)
    for name in ("lc_api.hip", "lc_internal.h"):
        text = open(os.path.join(CSRC, name)).read().replace("../../include/", os.path.join(ROOT, "include") + "/")
        (tmp_path / name).write_text(text)
    (tmp_path / "main.cpp").write_text(MAIN.replace("SCENARIOS", globals()[scenarios]))
    exe = tmp_path / "calls"
    res = subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-pthread", "-I", str(tmp_path), str(tmp_path / "main.cpp"), "-o", str(exe)],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]
    env = dict(os.environ, LC_TUNE_ONE_REST="0") if scenarios == "GIVEN_UP" else {k: v for k, v in os.environ.items() if not k.startswith("LC_TUNE")}
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=30, env=env)
    assert run.returncode == 0 and "as expected" in run.stdout, run.stdout[-3000:]
