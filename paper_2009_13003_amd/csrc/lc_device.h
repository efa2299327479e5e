// Device-side helpers shared by the encode and the decode kernels (gfx950, wave64): wavefront
// reductions and scans, the fp32 delta, streaming loads, and the element types of the parameter arrays.
#pragma once
#include "lc_internal.h"

// Wavefronts per SIMD that a kernel's registers are to allow, at least and at most.  (Its source is compiled for the host as well, by
// tests, where there is no such attribute.)
#ifdef __HIP__
#define LC_WAVES_PER_SIMD(least, most) __attribute__((amdgpu_waves_per_eu(least, most)))
#else
#define LC_WAVES_PER_SIMD(least, most)
#endif

namespace lc {

typedef unsigned long long u64;
typedef uint32_t u32;

// ----------------------------------------------------------------------------- small helpers
__device__ __forceinline__ u32 lane_id() { return __lane_id(); }

// Running sums over the wavefront (all 64 lanes active): DPP shifts within rows of 16 lanes, then the row totals carried
// across (row_bcast), no LDS traffic; a restore's chunk starts with one, and six LDS round trips were 0.25 us of it.
__device__ __forceinline__ u32 wave_incl_scan(u32 v) {
    v += (u32)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);     // row_shr:1
    v += (u32)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);     // row_shr:2
    v += (u32)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);     // row_shr:4
    v += (u32)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);     // row_shr:8
    v += (u32)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);     // row_bcast:15 into rows 1, 3
    v += (u32)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);     // row_bcast:31 into rows 2, 3
    return v;
}


// A word of memory that no kernel now running writes (tables and lists a previous kernel left), at an address that
// is the same in all lanes: read as constant memory it goes through the scalar cache, and waiting for it does not
// mean waiting for every vector load and store the wavefront has in flight.
__device__ __forceinline__ u32 load_uniform(const u32* p) {
    typedef const __attribute__((address_space(4))) u32* const_ptr;
    return *(const_ptr)(p);
}

// Where chunk c's entry lies in chunk_maxexp[kMaxChunks]: sweep 1 works on a window of consecutive chunks at any
// moment, and their atomics would all land in one or two cache lines (one memory channel); transposing the
// 512 x 512 index puts neighbouring chunks 2 KiB apart.
__device__ __forceinline__ u32 maxexp_slot(u32 c) {
    static_assert(kMaxChunks == 512u * 512u, "the transposition assumes 2^18 entries");
    return ((c & 511u) << 9) | (c >> 9);
}

// Largest value over the wavefront (all 64 lanes active), in every lane: row-wise running maxima with DPP
// shifts, then the row results carried across rows (row_bcast), no LDS traffic.
__device__ __forceinline__ u32 wave_max_u32(u32 v) {
    v = max(v, (u32)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false));     // row_shr:1
    v = max(v, (u32)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false));     // row_shr:2
    v = max(v, (u32)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false));     // row_shr:4
    v = max(v, (u32)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false));     // row_shr:8
    v = max(v, (u32)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false));     // row_bcast:15 into rows 1, 3
    v = max(v, (u32)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false));     // row_bcast:31 into rows 2, 3
    return (u32)__builtin_amdgcn_readlane((int)v, 63);
}

// Value of one lane (the same index in every lane), in every lane.
__device__ __forceinline__ u32 read_lane(u32 v, u32 l) { return (u32)__builtin_amdgcn_readlane((int)v, (int)l); }
__device__ __forceinline__ u64 read_lane64(u64 v, u32 l) { return ((u64)read_lane((u32)(v >> 32), l) << 32) | read_lane((u32)v, l); }

// The value of lane l, which may differ from lane to lane.
__device__ __forceinline__ u32 gather_lane(u32 v, u32 l) { return (u32)__shfl((int)v, (int)l, 64); }

// Canonical codes by one wavefront, lane j < 16 holding the length of symbol j (0: none): a code, left-justified, is the sum
// of the shares of the code space of the symbols before it, shorter ones first and by index within a length.  Each row of 16
// lanes takes a quarter of the symbols that may come before.  (lanes 16 and up: nothing)
__device__ __forceinline__ u32 canonical_code(u32 len) {
    const u32 lane = lane_id(), j = lane & 15;
    const u32 place = len ? len * 16 + lane : 0xFFFFu;
    const u32 mine = gather_lane(place, j);
    u32 before[4], sum = 0;
#pragma unroll
    for (u32 r = 0; r < 4; ++r) before[r] = gather_lane(place, (lane >> 4) * 4 + r);
#pragma unroll
    for (u32 r = 0; r < 4; ++r) sum += before[r] < mine ? 0x8000u >> (before[r] >> 4) : 0u;
    sum += __shfl_xor(sum, 16, 64);
    sum += __shfl_xor(sum, 32, 64);
    return len ? sum >> (15 - len) : 0u;
}

__device__ __forceinline__ u32 wave_sum32(u32 v) { return read_lane(wave_incl_scan(v), kW - 1); }

// (by pieces of 16 bits, whose sums fit 32: no LDS round trips)
__device__ __forceinline__ u64 wave_sum64(u64 v) {
    const u64 s0 = wave_sum32((u32)v & 0xFFFFu), s1 = wave_sum32((u32)v >> 16), s2 = wave_sum32((u32)(v >> 32) & 0xFFFFu), s3 = wave_sum32((u32)(v >> 48));
    return s0 + (s1 << 16) + (s2 << 32) + (s3 << 48);
}

// delta of Algorithm 1 line 4: one IEEE binary32 subtraction (never fused or reassociated).
__device__ __forceinline__ u32 delta_bits(float w, float w_ref) { return __float_as_uint(__fsub_rn(w, w_ref)); }
// ... and for binary64 parameters one binary64 subtraction
__device__ __forceinline__ u64 delta_bits(double w, double w_ref) { return (u64)__double_as_longlong(__dsub_rn(w, w_ref)); }

// 16-byte load of data that is read once: marked non-temporal so that the stream does not push
// other lines out of the caches (measured: +10 % read bandwidth on the sweeps).
typedef float f32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 load_stream(const float4* p) {
    const f32x4 v = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p));
    return make_float4(v.x, v.y, v.z, v.w);
}

// ---- element types of the parameter arrays.  The method works on the fp32 delta (Algorithm 1 line 4):
// bf16 / fp16 parameters are widened exactly on load, and the restored value fl32(w_ref + rep) is rounded
// once, to nearest even, on store.  Raw<DT> is what one lane holds of one row: 4 consecutive elements.
// binary64 parameters are coded on the binary64 delta, with 2^12 buckets (Section 3.1.1, footnote on the bucket
// count); Val<DT> is the type the arithmetic runs in, Bits<DT> its bit pattern.
struct Row64 { double x[4]; };
template <int DT> struct Raw { typedef uint2 type; };
template <> struct Raw<kF32> { typedef float4 type; };
template <> struct Raw<kF64> { typedef Row64 type; };
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
template <int DT> struct Val { typedef float type; typedef u32 bits; };
template <> struct Val<kF64> { typedef double type; typedef u64 bits; };

template <int DT> __device__ __forceinline__ constexpr u32 elem_bytes() { return DT == kF32 ? 4u : DT == kF64 ? 8u : 2u; }
template <int DT> __device__ __forceinline__ constexpr u32 exp_bits() { return DT == kF64 ? 11u : 8u; }
template <int DT> __device__ __forceinline__ constexpr u32 num_buckets() { return 2u << exp_bits<DT>(); }
// bucket id (sign and exponent bits) and biased exponent of a delta's bit pattern
__device__ __forceinline__ u32 bucket_of(u32 u) { return u >> 23; }
__device__ __forceinline__ u32 bucket_of(u64 u) { return (u32)(u >> 52); }

// 4 consecutive elements starting at element index i (a multiple of 4, base aligned to 4 elements), non-temporal
template <int DT>
__device__ __forceinline__ typename Raw<DT>::type load_raw(const void* base, u64 i) {
    if constexpr (DT == kF32) {
        return load_stream(reinterpret_cast<const float4*>(static_cast<const float*>(base) + i));
    } else {
        static_assert(DT != kF64, "binary64 rows: load_raw_any");
        const u32x2 v = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(static_cast<const uint16_t*>(base) + i));
        return make_uint2(v.x, v.y);
    }
}

// The same for an array that is aligned to its elements only: the hardware takes vectors at any address.
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef f32x4 __attribute__((aligned(4))) f32x4_any;
typedef u32x2 __attribute__((aligned(2))) u32x2_any;
typedef f64x2 __attribute__((aligned(8))) f64x2_any;
template <int DT, bool STREAM = true>            // STREAM false (binary64): plain loads
__device__ __forceinline__ typename Raw<DT>::type load_raw_any(const void* base, u64 i) {
    if constexpr (DT == kF32) {
        const f32x4 v = __builtin_nontemporal_load(reinterpret_cast<const f32x4_any*>(static_cast<const float*>(base) + i));
        return make_float4(v.x, v.y, v.z, v.w);
    } else if constexpr (DT == kF64) {
        const f64x2_any* p = reinterpret_cast<const f64x2_any*>(static_cast<const double*>(base) + i);
        if constexpr (!STREAM) { const f64x2 a = p[0], b = p[1]; return Row64{{a.x, a.y, b.x, b.y}}; }
        const f64x2 a = __builtin_nontemporal_load(p), b = __builtin_nontemporal_load(p + 1);
        return Row64{{a.x, a.y, b.x, b.y}};
    } else {
        const u32x2 v = __builtin_nontemporal_load(reinterpret_cast<const u32x2_any*>(static_cast<const uint16_t*>(base) + i));
        return make_uint2(v.x, v.y);
    }
}

__device__ __forceinline__ float widen16(u32 h, bool bf16) {
    return bf16 ? __uint_as_float(h << 16) : (float)__builtin_bit_cast(_Float16, (unsigned short)h);
}
__device__ __forceinline__ u32 narrow16(float x, bool bf16) {      // finite x, round to nearest even
    if (bf16) { const u32 u = __float_as_uint(x); return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16; }
    return (u32)__builtin_bit_cast(unsigned short, (_Float16)x);      // v_cvt_f16_f32, round to nearest even
}

// Two values at once, a in the low half.  bf16: v_cvt_pk_bf16_f32, which rounds every finite binary32 value as the
// integer formula above does (compared over all 2^32 patterns); infinities stay infinities.
typedef __bf16 lc_bf16x2 __attribute__((ext_vector_type(2)));
typedef float lc_f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u32 narrow16_pair(float a, float b, bool bf16) {
    if (bf16) { const lc_f32x2 f = {a, b}; return __builtin_bit_cast(u32, __builtin_convertvector(f, lc_bf16x2)); }
    return narrow16(a, false) | (narrow16(b, false) << 16);
}

__device__ __forceinline__ void unpack64(const Row64& r, double (&x)[4]) {
#pragma unroll
    for (int v = 0; v < 4; ++v) x[v] = r.x[v];
}

template <int DT>
__device__ __forceinline__ void unpack(const typename Raw<DT>::type& r, float (&x)[4]) {
    if constexpr (DT == kF32) { x[0] = r.x; x[1] = r.y; x[2] = r.z; x[3] = r.w; }
    else {
        x[0] = widen16(r.x & 0xFFFFu, DT == kBF16); x[1] = widen16(r.x >> 16, DT == kBF16);
        x[2] = widen16(r.y & 0xFFFFu, DT == kBF16); x[3] = widen16(r.y >> 16, DT == kBF16);
    }
}

// x as it reads back after a store in the storage type (rounded to nearest even; binary32: x itself)
template <int DT>
__device__ __forceinline__ float stored(float x) {
    if constexpr (DT == kF32) return x;
    else return widen16(narrow16(x, DT == kBF16), DT == kBF16);
}

template <int DT>
__device__ __forceinline__ float load_one(const void* base, u64 i) {
    if constexpr (DT == kF32) return static_cast<const float*>(base)[i];
    else return widen16(static_cast<const uint16_t*>(base)[i], DT == kBF16);
}

template <int DT>
__device__ __forceinline__ void store_one(void* base, u64 i, float x) {
    if constexpr (DT == kF32) static_cast<float*>(base)[i] = x;
    else static_cast<uint16_t*>(base)[i] = (uint16_t)narrow16(x, DT == kBF16);
}

// A row of 2-byte elements, aligned to 8 bytes, by a plain store (the sweep over several blobs, see fused_row).
template <int DT>
__device__ __forceinline__ void store4(void* base, u64 i, const float (&x)[4]) {
    static_assert(elem_bytes<DT>() == 2, "2-byte elements");
    *reinterpret_cast<u32x2*>(static_cast<uint16_t*>(base) + i) = u32x2{narrow16_pair(x[0], x[1], DT == kBF16), narrow16_pair(x[2], x[3], DT == kBF16)};
}

// Restored rows are written once and not read again by the sweep: non-temporal stores, like the loads (a bare
// read-modify-write sweep in this access pattern runs 4-5 % faster with both marked than with the loads alone).  The array may be
// aligned to its elements only.
template <int DT>
__device__ __forceinline__ void store4_any(void* base, u64 i, const typename Val<DT>::type (&x)[4]) {
    if constexpr (DT == kF32) {
        const f32x4 v = {x[0], x[1], x[2], x[3]};
        __builtin_nontemporal_store(v, reinterpret_cast<f32x4_any*>(static_cast<float*>(base) + i));
    } else if constexpr (DT == kF64) {
        // (plain stores: marked non-temporal, the two 16-byte halves of a lane's 32 bytes made the restore 15 % slower)
        f64x2_any* p = reinterpret_cast<f64x2_any*>(static_cast<double*>(base) + i);
        p[0] = f64x2{x[0], x[1]}; p[1] = f64x2{x[2], x[3]};
    } else {
        const u32x2 v = {narrow16_pair(x[0], x[1], DT == kBF16), narrow16_pair(x[2], x[3], DT == kBF16)};
        __builtin_nontemporal_store(v, reinterpret_cast<u32x2_any*>(static_cast<uint16_t*>(base) + i));
    }
}

// a row that may end inside, by elements, of binary64 parameters
__device__ __forceinline__ void load_row64(const void* __restrict__ p, u64 idx, u64 n, double (&x)[4]) {
#pragma unroll
    for (int v = 0; v < 4; ++v) x[v] = (idx + v < n) ? static_cast<const double*>(p)[idx + v] : 0.0;
}

template <bool FAST, int DT = kF32>
__device__ __forceinline__ void load_row(const void* __restrict__ p, u64 idx, u64 n, float (&x)[4]) {
    if (FAST) {
        unpack<DT>(load_raw<DT>(p, idx), x);
    } else {
#pragma unroll
        for (int v = 0; v < 4; ++v) x[v] = (idx + v < n) ? load_one<DT>(p, idx + v) : 0.0f;
    }
}

template <int DT, bool STREAM = true>
__device__ __forceinline__ void load_row_any(const void* __restrict__ p, u64 idx, typename Val<DT>::type (&x)[4]) {
    if constexpr (DT == kF64) unpack64(load_raw_any<kF64, STREAM>(p, idx), x);
    else unpack<DT>(load_raw_any<DT>(p, idx), x);
}

// ---- the same accesses and the restoring addition for any element type, on the type the arithmetic runs in
template <int DT>
__device__ __forceinline__ void load_row_v(const void* __restrict__ p, u64 idx, u64 n, typename Val<DT>::type (&x)[4]) {
    if constexpr (DT == kF64) load_row64(p, idx, n, x);
    else load_row<false, DT>(p, idx, n, x);
}
template <int DT>
__device__ __forceinline__ typename Val<DT>::type load_one_v(const void* base, u64 i) {
    if constexpr (DT == kF64) return static_cast<const double*>(base)[i];
    else return load_one<DT>(base, i);
}
template <int DT>
__device__ __forceinline__ void store_one_v(void* base, u64 i, typename Val<DT>::type x) {
    if constexpr (DT == kF64) static_cast<double*>(base)[i] = x;
    else store_one<DT>(base, i, x);
}
// Algorithm 1 line 7: one IEEE addition in the parameters' arithmetic type (never fused or reassociated)
__device__ __forceinline__ float add_rn(float a, float b) { return __fadd_rn(a, b); }
__device__ __forceinline__ double add_rn(double a, double b) { return __dadd_rn(a, b); }

// ---- what the kernels share that take codes apart (lc_decode.hip, lc_decode_one.hip)
__device__ __forceinline__ void raise_status(Workspace* ws, HostResult* host, u64 epoch, u32 status) {
    const u64 word = (epoch << 8) | status;
    atomicMax(&ws->dec_status, word);     // gates the decode sweep on the device
    host->dec_status = word;              // what the host reads after waiting for the stream (any finding will do)
}

// Symbol j of a blob, held by lane j of a wavefront.
struct DecSymbol { u32 len, code, rep, rep_hi; };

// By one wavefront: validates the header's symbol table and builds the canonical codes.  Returns (in every lane) whether it passes.
__device__ __forceinline__ bool dec_symbols(const u32* hdr, u64 n, u32 nchunks, u64 tw, DecSymbol* mine) {
    const u32 nbits = hdr[4], K = hdr[5], lane = lane_id();
    // binary64 blobs (element type 3): 12-bit bucket ids, 64-bit representatives with the high halves at offset 320
    const bool wide = hdr[15] == (u32)kF64;
    const u32 emask = wide ? 2047u : 255u, nbuckets = 2 * (emask + 1);
    bool ok = nbits >= 1 && nbits <= 4 && K <= (1u << nbits) - 1 && hdr[6] == kW && hdr[7] == kV && hdr[8] == kR;
    if (nchunks == 0 && tw != 0) ok = false;
    u32 len = 0, rep = 0, rep_hi = 0;
    u64 cn = 0;
    bool bad = false;
    if (ok && lane <= K) {
        const u32 j = lane, w0 = hdr[16 + 4 * j], bucket = w0 & 0xFFFFu;
        rep = hdr[17 + 4 * j]; rep_hi = wide ? hdr[80 + j] : 0u;
        cn = hdr[18 + 4 * j] | ((u64)hdr[19 + 4 * j] << 32);
        len = (w0 >> 16) & 0xFFu;
        if ((cn > 0) != (len > 0) || len > 15 || (w0 >> 24) != 0) { bad = true; len = 0; }
        if (j < K && (bucket >= nbuckets || (bucket & emask) == 0 || (bucket & emask) == emask)) bad = true;
        if (j < K && (wide ? (rep_hi >> 20) : (rep >> 23)) != bucket) bad = true;
        if (j == K && (rep | rep_hi) != 0) bad = true;
    }
    // (counts that add up to n modulo 2^64, as one running sum would have it)
    const u64 cnt_sum = wave_sum64(cn);
    const u32 kraft = wave_sum32(len ? 1u << (15 - len) : 0u), active = (u32)__popcll(__ballot(len != 0));
    if (ok && (__any(bad) || cnt_sum != n || (active >= 2 && kraft != (1u << 15)) || (active == 1 && kraft != (1u << 14)))) ok = false;
    mine->len = len; mine->code = canonical_code(len); mine->rep = rep; mine->rep_hi = rep_hi;
    return ok;
}

// A code, left-justified, is the largest of those not above a window that starts with it: code, length and symbol of lane j <
// 16, so that they compare in that order.
__device__ __forceinline__ u32 code_key(u32 len, u32 code) { return len ? (code << (15 - len)) << 8 | len << 4 | (lane_id() & 15u) : 0xFFFFFFFFu; }

// The sweeps' tables, by a workgroup of THREADS threads.  One symbol per look-up over the next 10 bits in `one`: symbol | len << 4;
// a prefix that starts no code: kOneNone; a prefix of a code longer than 10 bits: 0xFF.  From it every entry of
// the table of several symbols is then put together by taking codes off the front of its 10 bits, a thread's entries
// side by side (none: the entry of a prefix that starts no code).  ends (or null): bit b of an entry: one of its codes ends with
// bit b.  len, code: of symbol (lane) in every wavefront.  (Every dependent step here is latency of the call.)  Contains a barrier.
constexpr u32 kOneNone = 0xF0;
template <u32 THREADS>
__device__ __forceinline__ void dec_build_multi(u32* multi, uint8_t* one, uint16_t* ends, u32 none, u32 len, u32 code, u32 t) {
    constexpr u32 kEach = (1u << kMultiBits) / THREADS;
    const u32 key = code_key(len, code);
    u32 e[kEach];
#pragma unroll
    for (u32 k = 0; k < kEach; ++k) e[k] = 0;
#pragma unroll
    for (u32 j = 0; j < kMaxSym; ++j) {
        const u32 kj = read_lane(key, j);
#pragma unroll
        for (u32 k = 0; k < kEach; ++k) {
            const u32 at = ((t + THREADS * k) << (15 + 8 - kMultiBits)) | 0xFFu;
            e[k] = max(e[k], kj <= at ? kj : 0u);
        }
    }
#pragma unroll
    for (u32 k = 0; k < kEach; ++k) {
        const u32 at = (t + THREADS * k) << (15 - kMultiBits), L = (e[k] >> 4) & 15u;
        const bool starts = L != 0 && at < (e[k] >> 8) + (0x8000u >> L);
        e[k] = L > kMultiBits ? 0xFFu : starts ? e[k] & 0xFFu : kOneNone;
        one[t + THREADS * k] = (uint8_t)e[k];
    }
    __syncthreads();
    // (a prefix that gives no code, and a code longer than what is left, stop an entry for good: the same look-up again)
    u32 rest[kEach], left[kEach], syms[kEach], cnt[kEach], end[kEach];
#pragma unroll
    for (u32 k = 0; k < kEach; ++k) { rest[k] = (t + THREADS * k) << (32 - kMultiBits); left[k] = kMultiBits; syms[k] = 0; cnt[k] = 0; end[k] = 0; }
#pragma unroll
    for (u32 s = 0; s < kMultiSyms; ++s) {
        u32 f[kEach];
#pragma unroll
        for (u32 k = 0; k < kEach; ++k) f[k] = s == 0 ? e[k] : one[rest[k] >> (32 - kMultiBits)];
#pragma unroll
        for (u32 k = 0; k < kEach; ++k) {
            const u32 L = f[k] >> 4 <= left[k] ? f[k] >> 4 : 0u;
            syms[k] |= L ? (f[k] & 15u) << (4 * s) : 0u;
            cnt[k] += L ? 1u : 0u;
            rest[k] <<= L; left[k] -= L;
            end[k] |= 1u << (kMultiBits - left[k]);
        }
    }
#pragma unroll
    for (u32 k = 0; k < kEach; ++k) {
        const u32 i = t + THREADS * k;
        multi[i] = e[k] == kOneNone ? none : syms[k] | ((kMultiBits - left[k]) << 24) | (cnt[k] << 28);
        if (ends) ends[i] = (uint16_t)end[k];
    }
}

constexpr u32 kSparseSlack = 1024;   // bits above an all-merged chunk up to which a chunk's kept symbols are restored one by one
                                     // (512 instead: a batch of 2^24 elements at 2 bits 49 us, 40 so; 2048: the same)
constexpr u32 kSparseLaneSlack = 64; // the same for one lane's string

struct DecLds {
    alignas(16) u32 multi[1u << kMultiBits];
    float rep[kMaxSym];
    // the codes of more than 10 bits: symbol | len << 4 at [the next 15 bits - long_base].  They are the last codes in
    // canonical order, so the windows that start with one are the top of the 15-bit range; the code being complete, each
    // 10-bit prefix among those holds at least two of the 16 symbols, so there are at most 8 such prefixes
    alignas(4) uint8_t longs[8u << (15 - kMultiBits)];
    u32 long_base;
    double rep64[kMaxSym];            // binary64 blobs: the representatives (rep is not used then)
    template <int DT> __device__ __forceinline__ typename Val<DT>::type rep_of(u32 sy) const {
        if constexpr (DT == kF64) return rep64[sy];
        else return rep[sy];
    }
};

// the one symbol of a window whose first code is longer than the table's 10 bits, as an entry of the table
template <typename LDS>
__device__ __forceinline__ u32 decode_long(const LDS& L, u64 win) {
    const u32 e = L.longs[((u32)(win >> (64 - 15)) - L.long_base) & (sizeof(L.longs) - 1)];
    return (e & 15u) | ((e >> 4) << 24) | (1u << 28);
}

// That table, by one wavefront, lane j holding the length and code of symbol j (0 in lanes without one): 4 entries per lane.
// (A search through the symbols instead, a dependent look-up each, was most of a restore's time where such codes are
// many: 2^24 fp32 elements of 10 layers at 4 bits 193 us, 71 with the table.)
template <typename LDS>
__device__ __forceinline__ void build_longs(LDS& L, u32 len, u32 code) {
    const u32 base = 0x8000u - wave_max_u32(len > kMultiBits ? 0x8000u - (code << (15 - len)) : 0u);
    static_assert(sizeof(L.longs) == 4 * kW, "four entries per lane");
    u32 e[4] = {0, 0, 0, 0};                       // (nothing decodes to these: the windows past the last code do not exist)
    for (u64 m = __ballot(len > kMultiBits); m != 0; m &= m - 1) {
        const u32 j = (u32)__builtin_ctzll(m), lj = read_lane(len, j), cj = read_lane(code, j);
#pragma unroll
        for (u32 k = 0; k < 4; ++k) if (((base + 4 * lane_id() + k) >> (15 - lj)) == cj) e[k] = j | (lj << 4);
    }
    reinterpret_cast<u32*>(L.longs)[lane_id()] = e[0] | (e[1] << 8) | (e[2] << 16) | (e[3] << 24);
    if (lane_id() == 0) L.long_base = base;
}

// MSB-first bit window over payload words that live in LDS (STAGED) or in global memory.
template <bool STAGED>
struct BitReader {
    const u32* pw;                   // payload words (index 0 = first word of the chunk's payload)
    u32 last;                        // index of the last payload word (reads are clamped to it)
    u64 win;                         // next bits, left aligned
    u32 avail, wi, next;             // valid bits in win; index of `next`; the word after the window
    __device__ __forceinline__ u32 word(u32 i) const { return pw[min(i, last)]; }
    __device__ __forceinline__ void start(const u32* words, u32 nwords, u32 first_bit) {
        pw = words; last = nwords - 1;
        wi = first_bit >> 5;
        const u32 sh = first_bit & 31;
        win = (((u64)word(wi) << 32) | word(wi + 1)) << sh;
        avail = 64 - sh;
        wi += 2;
        next = word(wi);
    }
    __device__ __forceinline__ void refill() {           // leaves at least 33 valid bits
        if (avail <= 32) {
            win |= (u64)next << (32 - avail);
            avail += 32; ++wi;
            next = word(wi);
        }
    }
    __device__ __forceinline__ void drop(u32 len) { win <<= len; avail -= len; }
};

// ---- host-side helpers of the launchers
// Work items dealt round-robin to at most `cap` workers: the smallest worker count that keeps the number of
// rounds, so that every worker has the same load (+-1) and nobody idles through a last, half-empty round.
static inline uint64_t balanced_workers(uint64_t items, uint64_t cap) {
    if (items <= cap || cap == 0) return items;
    const uint64_t rounds = (items + cap - 1) / cap;
    return (items + rounds - 1) / rounds;
}

}  // namespace lc
