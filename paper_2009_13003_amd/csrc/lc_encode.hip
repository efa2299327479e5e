// Encode kernels of the LC-Checkpoint compress / restore path for gfx950 (wave64).
//
// lc_encode:         k_hist -> k_table -> k_pack -> k_place (whose first workgroup writes the header) (which also clears the scratch
//                    state for the next call, k_place the per-chunk maxima); k_reset only for a fresh scratch area
//                    (fp64 parameters: k_hist64 -> k_table<11> -> k_pack64 -> k_place)
//                    with staged keys: k_hist<..., KEYS> -> k_table -> k_pack_keys -> k_place
// lc_encode_cached:  k_spec_table -> k_spec_sweep -> k_table -> k_pack (nothing to do on a hit) -> k_place
// both, of a short vector (fp32, bf16, fp16) that the caller waits for: k_encode_one; k_reset_one behind one that was given up
// lc_encode_batch:   kb_setup -> kb_hist -> kb_table -> kb_list (long lists) -> kb_pack -> kb_place (whose first workgroups write the headers)
//
// The paper (arXiv 2009.13003) defines what is computed: delta against the last
// recovered state (Algorithm 1 line 4), (sign, exponent) buckets represented by the
// mean of their extremes and x-bit priority promotion (Section 3.1.1), Huffman
// coding of the bucket indices (Section 3.1.2).  How it is laid out on the GPU is this library's own.
#include "lc_meeting.h"
#include <stddef.h>
#include <type_traits>

namespace lc {

// ----------------------------------------------------------------------------- k_reset
// Brings the scratch state to what every encode call expects to find (and leaves behind):
// zero bucket counts, empty extremes, zero group sums and per-chunk exponent maxima.  Only launched
// for a fresh scratch area or after a call that did not run to its end.
__device__ __forceinline__ void clear_extremes(EncState* ws, u32 tid, u32 nthr) {
    u32* mn = &ws->mmin[0][0]; u32* mx = &ws->mmax[0][0];            // all copies
    for (u32 i = tid; i < kExtCopies * kMaxSym; i += nthr) { mn[i] = 0x7FFFFFu; mx[i] = 0; }
}

__device__ __forceinline__ void clear_encode_state(EncState* ws, u32* group_words, u32 ngroups, u32 tid, u32 nthr) {
    for (u32 i = tid; i < ngroups; i += nthr) group_words[i] = 0;
    clear_extremes(ws, tid, nthr);
    if (tid == 0) { ws->spec = 0; ws->spec_ok = 0; ws->list_count = 0; }
}

__device__ __forceinline__ void clear_ext64(Ext64* ext, u32 tid, u32 nthr) {
    for (u32 i = tid; i < kBuckets64; i += nthr) ext->hist[i] = 0;
    if (tid < kMaxSym) { ext->mmin[tid] = 0xFFFFFFFFFFFFFull; ext->mmax[tid] = 0; }
}

__device__ __forceinline__ void clear_bucket_extremes(Workspace* ws, u32 tid, u32 nthr) {
    for (u32 i = tid; i < 512; i += nthr) { ws->bucket_min[i] = 0xFFFFFFFFu; ws->bucket_max[i] = 0; }
}

__global__ void k_reset(Workspace* ws, u32* group_words, u32 ngroups, u32* chunk_maxexp, u32 nchunks) {
    clear_encode_state(ws, group_words, ngroups, threadIdx.x, blockDim.x);
    clear_ext64(&ws->ext64, threadIdx.x, blockDim.x);
    clear_bucket_extremes(ws, threadIdx.x, blockDim.x);
    for (u32 i = threadIdx.x; i < 512; i += blockDim.x) ws->hist[i] = 0;       // (where k_encode_one's workgroups meet)
    for (u32 i = threadIdx.x; i < nchunks; i += blockDim.x) chunk_maxexp[i] = 0;
}

// The same for a scratch area that only ever serves calls of at most `nchunks` chunks (their entries of the
// transposed maxima, their groups of 64 chunks): what such an area needs cleared before every call of its own.
__global__ void k_reset_chunks(Workspace* ws, u32* group_words, u32 ngroups, u32* chunk_maxexp, u32 nchunks) {
    clear_encode_state(ws, group_words, ngroups, threadIdx.x, blockDim.x);
    clear_ext64(&ws->ext64, threadIdx.x, blockDim.x);
    for (u32 c = threadIdx.x; c < nchunks; c += blockDim.x) chunk_maxexp[maxexp_slot(c)] = 0;
}

// What a call in one launch (k_encode_one, k_decode_one) leaves behind that was given up or refused.
__global__ void k_reset_one(Workspace* ws) {
    for (u32 i = threadIdx.x; i < 512; i += blockDim.x) ws->hist[i] = 0;       // (where the workgroups meet)
    clear_ext64(&ws->ext64, threadIdx.x, blockDim.x);
    clear_extremes(ws, threadIdx.x, blockDim.x);
}

// ----------------------------------------------------------------------------- k_hist
// Sweep 1 (Section 3.1.1, exponent-based quantization): population of each of the 2^9
// (sign, exponent) buckets.  LDS histogram replicated 8 times (copy = lane & 7, copies
// of one bin in different banks) so that lanes hitting the same popular bucket rarely
// collide; merged into 64-bit global counters once per workgroup (one of kHistCells copies of them).
constexpr int kHistCopies = 8;

// One 16-byte unit = EPU consecutive elements (4 fp32, 8 bf16 / fp16): counting does not care which lane
// sees which element, so every type is read in 16-byte accesses and kept as loaded until it is counted.
template <int DT, int EPU>
__device__ __forceinline__ void unpack_unit(const float4& t, float (&x)[EPU]) {
    if constexpr (DT == kF32) { x[0] = t.x; x[1] = t.y; x[2] = t.z; x[3] = t.w; }
    else {
        const u32 q[4] = {__float_as_uint(t.x), __float_as_uint(t.y), __float_as_uint(t.z), __float_as_uint(t.w)};
#pragma unroll
        for (int k = 0; k < 4; ++k) { x[2 * k] = widen16(q[k] & 0xFFFFu, DT == kBF16); x[2 * k + 1] = widen16(q[k] >> 16, DT == kBF16); }
    }
}

// 16 bytes of either array, which may be aligned to its elements only: the hardware takes vectors at any address.  Off alignment,
// against 16 bytes put together from single elements in this sweep alone (laplace but for the heavy-tailed ones): fp32 2^24 78 -> 73
// us the call, 2^26 heavy-tailed 125 -> 112, 2^26 bf16 155 -> 153; aligned arrays the same to 1 %.
typedef f32x4 __attribute__((aligned(2))) f32x4_anywhere;
__device__ __forceinline__ float4 load_unit(const void* __restrict__ p, u64 unit) {
    const f32x4 v = __builtin_nontemporal_load(static_cast<const f32x4_anywhere*>(p) + unit);
    return make_float4(v.x, v.y, v.z, v.w);
}
// The same put together from 2-byte elements (see launch_hist).
__device__ __forceinline__ float4 load_unit_halves(const void* __restrict__ p, u64 unit) {
    const uint16_t* q = static_cast<const uint16_t*>(p) + unit * 8;
    return make_float4(__uint_as_float(q[0] | ((u32)q[1] << 16)), __uint_as_float(q[2] | ((u32)q[3] << 16)),
                       __uint_as_float(q[4] | ((u32)q[5] << 16)), __uint_as_float(q[6] | ((u32)q[7] << 16)));
}

// Largest magnitude among the EPU deltas of one unit and m (its exponent field is the largest biased exponent).
// A NaN may drop out of a floating-point maximum: a vector with such a delta is not coded at all
// (the table's status says so), and nobody looks at the chunk maxima then.
template <int EPU>
__device__ __forceinline__ float max_magnitude(const u32 (&u)[EPU], float m) {
#pragma unroll
    for (int v = 0; v < EPU; ++v) m = fmaxf(m, fabsf(__uint_as_float(u[v])));
    return m;
}

// Every wavefront takes batches of PF consecutive rows of 64 units (PF KiB of each array), so a batch lies in
// one chunk of the coding sweep and its largest exponent goes to chunk_maxexp with one atomic per batch.
// batch_max (or null) receives every whole batch's largest exponent as a byte of its own: the coding sweep then
// knows which parts of a chunk it has to read.
// A wavefront keeps the maxima of its last 64 batches in LDS and writes them out 64 at a time, one per lane: a
// global write after every batch, however small, holds back the loads issued behind it (both are counted, in
// order, by the one vector-memory counter) and cost the sweep 4 % of its rate.
// KEYS (binary32): the sweep also stages a 9-bit key per element of every whole batch -- the 16
// exponent bytes and the 16 sign bits of the 16 elements a lane holds of a batch, which are the lane's own elements of
// 4 rows of the coding sweep's chunk -- and, being then the only sweep that sees the mantissas, tracks the smallest and
// largest delta bit pattern of every bucket (Section 3.1.1: the representative is the mean of these two).
template <int DT, bool KEYS = false, bool HALVES = false>
__global__ __launch_bounds__(1024) void k_hist(const void* __restrict__ w, const void* __restrict__ w_ref,
                                               u64 n, Workspace* ws, u32* chunk_maxexp, uint8_t* batch_max, KeyPlanes keys) {
    __shared__ u32 h[512 * kHistCopies];
    __shared__ u32 mn[KEYS ? 512 * kHistCopies : 1], mx[KEYS ? 512 * kHistCopies : 1];
    __shared__ uint16_t pend[1024 / kW][kW];         // per wavefront: the maxima of its batches not yet written out
    static_assert(!KEYS || DT == kF32, "keys are staged for binary32 arrays only");
    constexpr int EPU = 16 / (int)elem_bytes<DT>();
    const u32 tid = threadIdx.x, nthr = blockDim.x;
    for (u32 i = tid; i < 512 * kHistCopies; i += nthr) { h[i] = 0; if (KEYS) { mn[i] = 0xFFFFFFFFu; mx[i] = 0; } }
    __syncthreads();
    const u32 copy = tid & (kHistCopies - 1);
    const u64 nu = n / EPU;
    // Batches of PF rows per wavefront, one batch in flight while the previous one is counted.
    constexpr int PF = 4;
    constexpr u32 kBatchUnits = PF * kW;
    static_assert(kChunk % (kBatchUnits * EPU) == 0, "a batch must not straddle two chunks");
    const u64 nbatch = nu / kBatchUnits;
    const u64 stride = (u64)gridDim.x * (nthr / kW);                    // wavefronts in the grid
    u64 b = (u64)blockIdx.x * (nthr / kW) + tid / kW;
    float4 a0[PF], b0[PF], a1[PF], b1[PF];
    auto fetch = [&](float4 (&a)[PF], float4 (&bb)[PF], u64 batch) {
        const u64 at = batch * kBatchUnits + (tid & (kW - 1));
#pragma unroll
        for (int k = 0; k < PF; ++k) {
            a[k] = HALVES ? load_unit_halves(w, at + k * kW) : load_unit(w, at + k * kW);
            bb[k] = HALVES ? load_unit_halves(w_ref, at + k * kW) : load_unit(w_ref, at + k * kW);
        }
    };
    u32 pending = 0;                                 // maxima waiting in pend, those of batches pend_first, + stride, ...
    u64 pend_first = b;
    auto write_maxima = [&]() {
        __builtin_amdgcn_wave_barrier();
        const u32 lane = tid & (kW - 1);
        if (lane < pending) {
            const u64 batch = pend_first + (u64)lane * stride;
            const u32 m = pend[tid / kW][lane];
            atomicMax(&chunk_maxexp[maxexp_slot((u32)((batch * kBatchUnits * EPU) / kChunk))], m);
            if (batch_max) batch_max[batch] = (uint8_t)m;
        }
        __builtin_amdgcn_wave_barrier();
    };
    u32 key_word = 0, key_signs = 0;                 // KEYS: exponent bytes of the unit just counted; sign bits of the batch so far
    auto count_one = [&](u32 u) {
        const u32 at = (u >> 23) * kHistCopies + copy;
        atomicAdd(&h[at], 1u);
        if (KEYS) { atomicMin(&mn[at], u); atomicMax(&mx[at], u); }
    };
    auto count_unit = [&](const float4& a, const float4& bb, float m) {
        float x[EPU], y[EPU];
        u32 u[EPU];
        unpack_unit<DT, EPU>(a, x); unpack_unit<DT, EPU>(bb, y);
        key_word = 0;
#pragma unroll
        for (int v = 0; v < EPU; ++v) {
            u[v] = delta_bits(x[v], y[v]);
            count_one(u[v]);
            if (KEYS) { key_word |= ((u[v] >> 23) & 255u) << (8 * v); key_signs = (key_signs >> 1) | ((u[v] >> 31) << 15); }
        }
        return max_magnitude<EPU>(u, m);
    };
    auto count = [&](float4 (&a)[PF], float4 (&bb)[PF], u64 batch) {
        float mf = 0.f;
        u32 kw[PF];
#pragma unroll
        for (int k = 0; k < PF; ++k) { mf = count_unit(a[k], bb[k], mf); kw[k] = key_word; }
        if constexpr (KEYS) {
            // (after 16 elements the sign bit of element 4 k + v has arrived at bit 4 k + v)
            static_assert(PF == 4 && EPU == 4, "a batch is 4 rows of 4 elements per lane");
            const u32x4 kv = {kw[0], kw[1], kw[2], kw[3]};
            const u64 at = batch * kW + (tid & (kW - 1));
            __builtin_nontemporal_store(kv, reinterpret_cast<u32x4*>(keys.exp) + at);
            __builtin_nontemporal_store((uint16_t)key_signs, keys.sign + at);
        }
        const u32 m = wave_max_u32(__float_as_uint(mf));     // whole wavefronts only: b < nbatch is the same for all lanes
        if ((tid & (kW - 1)) == 0) pend[tid / kW][pending] = (uint16_t)(m >> 23);
        if (++pending == kW) { write_maxima(); pending = 0; pend_first = batch + stride; }
    };
    if (b < nbatch) {
        // The loads of the batch after next are issued without a branch around them (at the end the current
        // batch is simply read again): only then does the compiler wait for the older batch alone.
        fetch(a0, b0, b);
        while (true) {
            const bool more1 = b + stride < nbatch;
            fetch(a1, b1, more1 ? b + stride : b);
            count(a0, b0, b);
            if (!more1) break;
            b += stride;
            const bool more0 = b + stride < nbatch;
            fetch(a0, b0, more0 ? b + stride : b);
            count(a1, b1, b);
            if (!more0) break;
            b += stride;
        }
        write_maxima();
    }
    // what is left of the vector: fewer than one batch of units, then fewer than one unit of elements
    if (blockIdx.x == 0) {
        for (u64 u = nbatch * kBatchUnits + tid; u < nu; u += nthr) {
            const float mf = count_unit(load_unit(w, u), load_unit(w_ref, u), 0.f);
            atomicMax(&chunk_maxexp[maxexp_slot((u32)((u * EPU) / kChunk))], __float_as_uint(mf) >> 23);
        }
        if (tid < (u32)(n - EPU * nu)) {
            const u64 i = EPU * nu + tid;
            const u32 u = delta_bits(load_one<DT>(w, i), load_one<DT>(w_ref, i));
            count_one(u);
            atomicMax(&chunk_maxexp[maxexp_slot((u32)(i / kChunk))], (u >> 23) & 255u);
        }
    }
    __syncthreads();
    for (u32 bk = tid; bk < 512; bk += nthr) {
        u32 sum = 0, lo = 0xFFFFFFFFu, hi = 0;
#pragma unroll
        for (int k = 0; k < kHistCopies; ++k) {
            sum += h[bk * kHistCopies + k];
            if (KEYS) { lo = min(lo, mn[bk * kHistCopies + k]); hi = max(hi, mx[bk * kHistCopies + k]); }
        }
        if (sum) {
            atomicAdd(&ws->ext64.hist[(blockIdx.x % kHistCells) * 512 + bk], (u64)sum);
            if (KEYS) { atomicMin(&ws->bucket_min[bk], lo); atomicMax(&ws->bucket_max[bk], hi); }
        }
    }
}

// ----------------------------------------------------------------------------- k_hist64
// Sweep 1 for binary64 parameters: the same walk over the arrays (a 16-byte unit holds 2 elements, a batch of 4 rows
// 512), 2^12 buckets (sign and 11 exponent bits; Section 3.1.1, footnote on the bucket count) in 2 LDS copies,
// counts and chunk maxima of the binary64 delta.
constexpr int kHistCopies64 = 2;

__global__ __launch_bounds__(1024) void k_hist64(const void* __restrict__ w, const void* __restrict__ w_ref,
                                                 u64 n, Ext64* ext, u32* chunk_maxexp, uint16_t* part_max) {
    __shared__ u32 h[kBuckets64 * kHistCopies64];
    __shared__ uint16_t pend[1024 / kW][kW];         // as in k_hist: maxima written out 64 batches at a time
    constexpr int EPU = 2;
    const u32 tid = threadIdx.x, nthr = blockDim.x;
    for (u32 i = tid; i < kBuckets64 * kHistCopies64; i += nthr) h[i] = 0;
    __syncthreads();
    const u32 copy = tid & (kHistCopies64 - 1);
    const u64 nu = n / EPU;
    constexpr int PF = 4;
    constexpr u32 kBatchUnits = PF * kW;
    static_assert(kChunk % (kBatchUnits * EPU) == 0, "a batch must not straddle two chunks");
    const u64 nbatch = nu / kBatchUnits;
    const u64 stride = (u64)gridDim.x * (nthr / kW);
    u64 b = (u64)blockIdx.x * (nthr / kW) + tid / kW;
    float4 a0[PF], b0[PF], a1[PF], b1[PF];
    auto fetch = [&](float4 (&a)[PF], float4 (&bb)[PF], u64 batch) {
        const u64 at = batch * kBatchUnits + (tid & (kW - 1));
#pragma unroll
        for (int k = 0; k < PF; ++k) { a[k] = load_unit(w, at + k * kW); bb[k] = load_unit(w_ref, at + k * kW); }
    };
    u32 pending = 0;
    u64 pend_first = b;
    // (a batch is 4 KiB of each array: the largest exponent of every such part lets sweep 2 read a mostly merged
    // chunk part by part, as for the other element types; 11 exponent bits: two bytes each)
    auto write_maxima = [&]() {
        __builtin_amdgcn_wave_barrier();
        const u32 lane = tid & (kW - 1);
        if (lane < pending) {
            const u64 batch = pend_first + (u64)lane * stride;
            const u32 m = pend[tid / kW][lane];
            atomicMax(&chunk_maxexp[maxexp_slot((u32)((batch * kBatchUnits * EPU) / kChunk))], m);
            if (part_max) part_max[batch] = (uint16_t)m;
        }
        __builtin_amdgcn_wave_barrier();
    };
    auto as_double = [](float lo, float hi) { return __hiloint2double(__float_as_int(hi), __float_as_int(lo)); };
    auto count_one = [&](double x, double y, u32 m) {       // returns the larger of m and the delta's biased exponent
        const u64 u = delta_bits(x, y);
        atomicAdd(&h[bucket_of(u) * kHistCopies64 + copy], 1u);
        return max(m, bucket_of(u) & 2047u);
    };
    auto count_unit = [&](const float4& a, const float4& bb, u32 m) {
        m = count_one(as_double(a.x, a.y), as_double(bb.x, bb.y), m);
        return count_one(as_double(a.z, a.w), as_double(bb.z, bb.w), m);
    };
    auto count = [&](float4 (&a)[PF], float4 (&bb)[PF], u64 batch) {
        u32 m = 0;
#pragma unroll
        for (int k = 0; k < PF; ++k) m = count_unit(a[k], bb[k], m);
        m = wave_max_u32(m);
        if ((tid & (kW - 1)) == 0) pend[tid / kW][pending] = (uint16_t)m;
        if (++pending == kW) { write_maxima(); pending = 0; pend_first = batch + stride; }
    };
    if (b < nbatch) {
        fetch(a0, b0, b);
        while (true) {
            const bool more1 = b + stride < nbatch;
            fetch(a1, b1, more1 ? b + stride : b);
            count(a0, b0, b);
            if (!more1) break;
            b += stride;
            const bool more0 = b + stride < nbatch;
            fetch(a0, b0, more0 ? b + stride : b);
            count(a1, b1, b);
            if (!more0) break;
            b += stride;
        }
        write_maxima();
    }
    if (blockIdx.x == 0) {
        for (u64 u = nbatch * kBatchUnits + tid; u < nu; u += nthr) {
            const u32 m = count_unit(load_unit(w, u), load_unit(w_ref, u), 0);
            atomicMax(&chunk_maxexp[maxexp_slot((u32)((u * EPU) / kChunk))], m);
        }
        if (tid < (u32)(n - EPU * nu)) {
            const u64 i = EPU * nu + tid;
            const u32 m = count_one(static_cast<const double*>(w)[i], static_cast<const double*>(w_ref)[i], 0);
            atomicMax(&chunk_maxexp[maxexp_slot((u32)(i / kChunk))], m);
        }
    }
    __syncthreads();
    for (u32 bk = tid; bk < kBuckets64; bk += nthr) {
        const u32 sum = h[bk * kHistCopies64] + h[bk * kHistCopies64 + 1];
        if (sum) atomicAdd(&ext->hist[bk], (u64)sum);
    }
}

// ----------------------------------------------------------------------------- k_table
// Priority promotion (Section 3.1.1) and the Huffman table (Section 3.1.2): one workgroup and, where a chain of single
// steps is left, its first wavefront.  Nothing here is bound by bytes; it is the latency of that chain, which every encode
// waits for.  So the buckets are ranked by all threads at once, and the chain keeps to scalar registers: see code_lengths.
// One wavefront with 64-bit weights, ranking included, against this: a 2^27 bf16 vector at 4 bits (with its list of chunks)
// 14.1 -> 8.6 us, 161 tensors 11.9 -> 5.1 us.
template <int EB>                         // EB: exponent bits of the parameters' delta (8, or 11 for binary64)
struct TableLds {
    alignas(8) uint8_t sym[2u << EB];     // bucket -> symbol, 0xFF: merged
    u64 cnt[kMaxSym];
    u32 kept[kMaxSym];
    u32 found[kW];                        // candidates among the buckets of one step of one wavefront, in order of rank
    u32 nonfinite, zero_class;
    uint8_t symlen[kMaxSym];              // symbol | length << 4; the last entry: the merged symbol's (there are at most 15 others)
};
template <int EB> constexpr u32 table_threads() { return EB == 8 ? 512u : 1024u; }
template <int EB> constexpr u32 table_steps() { return (2u << EB) / table_threads<EB>(); }

// Places of the buckets in order of priority: larger exponent first, + before - at equal exponent.
template <int EB> __device__ __forceinline__ u32 bucket_at(u32 i) { return ((i & 1u) << EB) | (((1u << EB) - 1) - (i >> 1)); }

// Ranks the non-empty normal buckets and fills S (all but symlen); thread t of table_threads holds the population of the
// bucket at place t + s * table_threads in c[s].  By a workgroup of at least that many threads (the others hold zeros);
// contains a barrier, and the caller's comes before S is read.  Returns the number of candidates.
template <int EB>
__device__ __forceinline__ u32 rank_buckets(TableLds<EB>& S, const u64 (&c)[table_steps<EB>()], u32 kmax) {
    constexpr u32 kThreads = table_threads<EB>(), kSteps = table_steps<EB>(), kWaves = kThreads / kW, kEmax = (1u << EB) - 1;
    static_assert(kSteps * kWaves <= kW, "one lane per count of the scan");
    const u32 t = threadIdx.x, lane = lane_id(), wave = t / kW;
    u64 m[kSteps];
#pragma unroll
    for (u32 s = 0; s < kSteps; ++s) {
        const u32 E = bucket_at<EB>(t + s * kThreads) & kEmax;
        const u64 any = __ballot(c[s] != 0);
        m[s] = __ballot(c[s] != 0 && E != 0 && E != kEmax);
        if (lane == 0 && t < kThreads) S.found[s * kWaves + wave] = (u32)__popcll(m[s]);
        // (the two buckets of infinities and NaN are places 0 and 1, those of zeros and subnormals the last two)
        if (s == 0 && t == 0) S.nonfinite = (any & 3u) != 0 ? 1u : 0u;
        if (s == kSteps - 1 && t == kThreads - 1) S.zero_class = (any >> (kW - 2)) != 0 ? 1u : 0u;
    }
    if (t < kMaxSym) { S.cnt[t] = 0; S.kept[t] = 0; }
    __syncthreads();
    const u32 mine = lane < kSteps * kWaves ? S.found[lane] : 0u, incl = wave_incl_scan(mine), excl = incl - mine;
    if (t < kThreads) {
#pragma unroll
        for (u32 s = 0; s < kSteps; ++s) {
            const u32 b = bucket_at<EB>(t + s * kThreads);
            const u32 r = read_lane(excl, __builtin_amdgcn_readfirstlane(s * kWaves + wave)) + (u32)__popcll(m[s] & ((1ull << lane) - 1));
            const bool keep = ((m[s] >> lane) & 1) != 0 && r < kmax;
            S.sym[b] = keep ? (uint8_t)r : (uint8_t)0xFF;
            if (keep) { S.kept[r] = b; S.cnt[r] = c[s]; }
        }
    }
    return read_lane(incl, kW - 1);
}

// The sum over lanes l, l ^ 16, l ^ 32 and l ^ 48, in all four (gfx950: rows and halves change places without LDS).
__device__ __forceinline__ u32 rows_sum(u32 v) {
    const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = a[0] + a[1];
    const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return b[0] + b[1];
}

// Huffman code lengths by one wavefront, lane j < 16 holding the count of symbol j (0: does not occur; so do the other lanes);
// at least two occur, and their counts add up to at most 2^32.  Repeatedly joins the two smallest nodes under the order
// (weight, leaf before joined node, symbol index / creation order) with two queues, both sorted: the leaves, moved to lanes
// 0 .. 15 in ascending order, and the joined nodes in creation order in lanes 32 and up.  The loop keeps to scalar registers
// and real branches (as selects its conditions took 410 cycles a turn, so 110).  A node remembers its parent only; the depths
// follow by doubling the step towards the root four times.  Weights of 32 bits are enough: a node that is ever
// compared leaves something out.
__device__ __forceinline__ u32 code_lengths(u32 count) {
    constexpr u32 kNone = 0xFFFFFFFFu, kNodes = 32;
    const u32 lane = lane_id(), j = lane & 15;
    const u32 nl = (u32)__popcll(__ballot(count != 0));
    // where each goes: how many come before it, a quarter of them counted in each row of 16 lanes (absent: behind all others)
    const u32 key = count - 1, mine = gather_lane(key, j);
    u32 other[4], place = 0;
#pragma unroll
    for (u32 r = 0; r < 4; ++r) other[r] = gather_lane(key, (lane >> 4) * 4 + r);
#pragma unroll
    for (u32 r = 0; r < 4; ++r) place += (other[r] < mine || (other[r] == mine && (lane >> 4) * 4 + r < j)) ? 1u : 0u;
    place = rows_sum(place);
    u32 w = (u32)__builtin_amdgcn_ds_permute((int)(place * 4), (int)(mine + 1));      // (four lanes write each, the same)
    if (lane >= nl) w = kNone;
    u32 parent = lane, li = 0, qi = kNodes, lw = read_lane(w, 0), nw = kNone;
#pragma unroll 1
    for (u32 ni = kNodes; ni < kNodes + nl - 1; ++ni) {
        u32 sum = 0;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            // (behind the last leaf and the last node there is nothing: kNone)
            if (lw <= nw) {
                asm volatile("");
                sum += lw; parent = lane == li ? ni : parent; ++li; lw = read_lane(w, li);
            } else {
                asm volatile("");
                sum += nw; parent = lane == qi ? ni : parent; ++qi; nw = read_lane(w, qi);
            }
        }
        w = lane == ni ? sum : w;
        if (qi == ni) nw = sum;                              // the queue of nodes was empty: its head
    }
    u32 depth = parent != lane ? 1u : 0u, up = parent;
#pragma unroll
    for (int k = 0; k < 4; ++k) {                            // (no symbol of 16 lies deeper than 15)
        const u32 d = gather_lane(depth, up), u = gather_lane(up, up);
        depth += d; up = u;
    }
    const u32 len = gather_lane(depth, place);
    return count != 0 ? len : 0u;
}

// The counts of the symbols, one per lane of a wavefront: the kept buckets' and, in lane K, what is left of n.
__device__ __forceinline__ u64 symbol_count(const u64* cnt, u32 K, u64 n) {
    const u32 lane = lane_id();
    const u64 c = lane < K ? cnt[lane] : 0ull;
    const u32 kept = wave_sum32((u32)c);                     // (modulo 2^32: n <= 2^32, and no kept bucket holds them all unless K > 0)
    const u64 rest = K == 0 ? n : (u64)((u32)n - kept);
    return lane == K ? rest : c;
}

// When the sweep before it coded speculatively with a cached table (ws->spec), the kernel also decides
// whether that stands: this checkpoint's kept set must be the cached one and exactly the symbols with a
// cached code must occur, in a coding of at most n * nbits payload bits.  If so the cached lengths are kept and the sweep's output is final (spec_ok);
// if not, the traces of the speculative coding are cleared and the table is this checkpoint's own.
// With chunk_list (and a workgroup of 1024 threads) the wavefronts but the first meanwhile list the chunks
// that sweep 2 has to read: all but the full chunks whose largest exponent lies below every kept bucket.
// (EB 8: the counts of a vector are CELLS copies in ext, those of a tensor of a batched call one array in its state)
template <int EB, u32 CELLS = 1>
__device__ __forceinline__ void table_build(EncState* ws, Ext64* ext, u64 n, int nbits, u32* group_words, u32 ngroups,
                                            const u32* chunk_maxexp, u32* chunk_list) {
    __shared__ TableLds<EB> S;
    constexpr u32 kEmax = (1u << EB) - 1, kThreads = table_threads<EB>(), kSteps = table_steps<EB>();
    const unsigned long long* hist = EB == 8 && CELLS == 1 ? ws->hist : ext->hist;
    __shared__ u32 s_reuse, s_listed;
    const u32 lane = lane_id(), t = threadIdx.x;
    const bool active = t < kW;
    const u32 kmax = (1u << nbits) - 1;
    u64 cnt[kSteps];
#pragma unroll
    for (u32 s = 0; s < kSteps; ++s) {
        u64 part[CELLS];
#pragma unroll
        for (u32 k = 0; k < CELLS; ++k) part[k] = t < kThreads ? hist[k * 512 + bucket_at<EB>(t + s * kThreads)] : 0;
        cnt[s] = 0;
#pragma unroll
        for (u32 k = 0; k < CELLS; ++k) cnt[s] += part[k];
    }
    const u32 spec = ws->spec;
    // The groups' record sizes start from zero in every call: the last call's placement read them to its end, so they
    // are cleared here, ahead of the coding sweep that adds to them (a cached table's speculative coding has already
    // added to them: then k_spec_table has cleared them).
    if (group_words && !spec) for (u32 i = t; i < ngroups; i += blockDim.x) group_words[i] = 0;
    // The other wavefronts list chunks; the maxima of their first batch are already on their way while the
    // buckets are ranked (a chunk with a ragged end is always read).  Work item t stands for
    // slot (hi << 9) | lo of the transposed maxima, hi = t / per_row, so that a wavefront's loads fall on a few
    // cache lines; its chunk is (lo << 9) | hi.  One batch covers the 16384 chunks of a 2^28-element call.
    constexpr u32 kListBatch = 18;
    const bool lister = chunk_list && t >= kW;
    const u32 workers = blockDim.x - kW, list_first = (t - kW) & ~(kW - 1);
    const u32 nchunks = (u32)num_chunks_of(n), nfull = (u32)(n / kChunk);
    const u32 per_row = nchunks > 512 ? (nchunks + 511) >> 9 : 1, items = 512 * per_row;
    const float inv_per_row = 1.0f / (float)per_row;
    u32 maxima[kListBatch], chunk_of[kListBatch];
    auto fetch_maxima = [&](u32 t0) {
#pragma unroll
        for (u32 u = 0; u < kListBatch; ++u) {
            const u32 t = t0 + u * workers + lane;
            u32 hi = (u32)((float)t * inv_per_row);                    // t < 2^18: off by one at most
            if (hi * per_row > t) --hi; else if ((hi + 1) * per_row <= t) ++hi;
            const u32 lo = t - hi * per_row, c = (lo << 9) | hi;
            chunk_of[u] = t < items ? c : 0xFFFFFFFFu;
            maxima[u] = (t < items && c < nfull) ? chunk_maxexp[(hi << 9) | lo] : 0xFFFFFFFFu;
        }
    };
    if (lister) fetch_maxima(list_first);
    const u32 total = rank_buckets<EB>(S, cnt, kmax), K = total < kmax ? total : kmax;
    if (t == 0) s_listed = 0;
    __syncthreads();
    const u32 min_kept_exp = K ? (S.kept[K - 1] & kEmax) : kEmax + 1;   // kept buckets are in descending exponent order
    if (lister) {
        for (u32 t0 = list_first; t0 < items; t0 += kListBatch * workers) {
            if (t0 != list_first) fetch_maxima(t0);
            u64 m[kListBatch];
            u32 found = 0;
#pragma unroll
            for (u32 u = 0; u < kListBatch; ++u) {
                m[u] = __ballot(chunk_of[u] < nchunks && maxima[u] >= min_kept_exp);
                found += (u32)__popcll(m[u]);
            }
            if (found == 0) continue;
            u32 base = 0;                                  // one claim on the list per batch
            if (lane == 0) base = atomicAdd(&s_listed, found);
            base = __builtin_amdgcn_readfirstlane(base);
#pragma unroll
            for (u32 u = 0; u < kListBatch; ++u) {
                if ((m[u] >> lane) & 1) chunk_list[base + __popcll(m[u] & ((1ull << lane) - 1))] = chunk_of[u];
                base += (u32)__popcll(m[u]);
            }
        }
    }
    if (active) {
        // The first wavefront builds the code; lane j holds what belongs to symbol j.
        Table& T = ws->table;
        const bool nonfinite = S.nonfinite != 0;
        const u64 c = symbol_count(S.cnt, K, n);
        const u32 msym = K + 1;
        const u32 nl = (u32)__popcll(__ballot(c != 0));
        u32 len = 0;
        bool reuse = false;
        if (spec) {
            bool differs = false;
            u32 cached_len = 0;
            if (lane < K) differs = T.kept[lane] != S.kept[lane];
            if (lane < msym) { cached_len = T.codelen[lane] & 31; differs = differs || ((cached_len != 0) != (c != 0)); }
            // ... and the cached lengths must not need more than the n * nbits payload bits every blob is promised to
            // fit (a stale table on shifted populations can; this checkpoint's own Huffman code never does)
            const u64 payload_bits = wave_sum64(lane < msym ? c * cached_len : 0ull);
            reuse = !nonfinite && T.K == K && !__any(differs) && payload_bits <= n * (u64)nbits;
            if (reuse) len = cached_len;
        }
        if (!reuse && nl == 1) len = c != 0 ? 1u : 0u;
        if (!reuse && nl >= 2) len = code_lengths((u32)c);
        const u32 code = canonical_code(len), max_len = wave_max_u32(len);
        if (lane < kMaxSym) {
            T.codelen[lane] = lane < msym ? ((code << 5) | len) : 0;
            T.kept[lane] = lane < K ? S.kept[lane] : 0;
            T.cnt[lane] = lane < msym ? c : 0;
            if (lane != kMaxSym - 1) S.symlen[lane] = (uint8_t)(lane | (len << 4));
        }
        if (lane == K) S.symlen[kMaxSym - 1] = (uint8_t)(lane | (len << 4));
        if (lane == 0) {
            s_reuse = reuse;
            ws->spec_ok = reuse;
            T.K = K; T.max_len = max_len; T.k_E = total + S.zero_class;
            T.min_kept_exp = min_kept_exp;
            T.status = nonfinite ? 2u : 0u;
        }
    }
    __syncthreads();
    if (t == 0) ws->list_count = s_listed;
    uint8_t* symlen_of_bucket = EB == 8 ? ws->table.symlen_of_bucket : ext->symlen_of_bucket;
    static_assert(offsetof(Table, symlen_of_bucket) % 8 == 0 && offsetof(Ext64, symlen_of_bucket) % 8 == 0, "8 buckets per store");
    for (u32 i = t; i < (2u << EB) / 8; i += blockDim.x) {
        const u64 sy = reinterpret_cast<const u64*>(S.sym)[i];
        u64 out = 0;
#pragma unroll
        for (u32 k = 0; k < 8; ++k) out |= (u64)S.symlen[(u32)(sy >> (8 * k)) & 15u] << (8 * k);     // (0xFF: the last entry)
        reinterpret_cast<u64*>(symlen_of_bucket)[i] = out;
    }
    if (active && spec && !s_reuse) {              // the speculative coding is void: forget its extremes and sizes
        for (u32 i = lane; i < ngroups; i += kW) group_words[i] = 0;
        clear_extremes(ws, lane, kW);
    }
}

template <int EB>
__global__ __launch_bounds__(1024) void k_table(EncState* ws, Ext64* ext, u64 n, int nbits, u32* group_words, u32 ngroups,
                                                 const u32* chunk_maxexp, u32* chunk_list) {
    table_build<EB, EB == 8 ? kHistCells : 1>(ws, ext, n, nbits, group_words, ngroups, chunk_maxexp, chunk_list);
}

// ----------------------------------------------------------------------------- k_spec_table
// lc_encode_cached, before the sweep: turns a usable cache (valid, same nbits, kept buckets in strict
// priority order, lengths forming a complete prefix code) into the table the sweep codes with.
template <int EB>                         // EB: exponent bits of the parameters' delta (8, or 11 for binary64)
__global__ __launch_bounds__(64) void k_spec_table(EncState* ws, Ext64* ext, const TableCache* cache, int nbits,
                                                   u32* group_words, u32 ngroups) {
    constexpr u32 kBuckets = 2u << EB, kEmax = (1u << EB) - 1;
    __shared__ u32 s_ok, s_len[kMaxSym + 1];
    __shared__ uint8_t s_sym[kBuckets];
    const u32 lane = threadIdx.x;
    Table& T = ws->table;
    for (u32 i = lane; i < ngroups; i += kW) group_words[i] = 0;      // (the sweep that follows may add to them: see k_table)
    for (u32 b = lane; b < kBuckets; b += kW) s_sym[b] = 0xFF;
    __syncthreads();
    if (lane == 0) {
        const u32 kmax = (1u << nbits) - 1, K = cache->K;
        bool ok = cache->valid == 1 && cache->nbits == (u32)nbits && K <= kmax;
        u32 kraft = 0, nact = 0, max_len = 0, per_len[17];
        for (int L = 0; L <= 16; ++L) per_len[L] = 0;
        for (u32 j = 0; j <= kMaxSym; ++j) s_len[j] = 0;
        if (ok) {
            u32 prev_key = 0xFFFFFFFFu;
            for (u32 j = 0; j < K; ++j) {
                const u32 b = cache->kept[j], e = b & kEmax;
                const u32 key = (e << 1) | (1u - ((b >> EB) & 1u));    // larger exponent first, + before -
                if (b >= kBuckets || e == 0 || e == kEmax || key >= prev_key) { ok = false; break; }
                prev_key = key;
            }
            for (u32 j = 0; j <= K && ok; ++j) {
                const u32 l = cache->len[j];
                if (l > 15) { ok = false; break; }
                s_len[j] = l;
                if (l) { kraft += 1u << (15 - l); ++nact; per_len[l]++; if (l > max_len) max_len = l; }
            }
            if (nact >= 2 && kraft != (1u << 15)) ok = false;
            if (nact == 1 && kraft != (1u << 14)) ok = false;
        }
        if (ok) {
            u32 next_code[17], code = 0;
            for (int L = 1; L <= 16; ++L) { code = (code + per_len[L - 1]) << 1; next_code[L] = code; }
            for (u32 j = 0; j < kMaxSym; ++j) {
                const u32 c = (j <= K && s_len[j]) ? next_code[s_len[j]]++ : 0;
                T.codelen[j] = j <= K ? ((c << 5) | s_len[j]) : 0;
                T.kept[j] = j < K ? cache->kept[j] : 0;
                T.cnt[j] = 0;
                if (j < K) s_sym[cache->kept[j]] = j;
            }
            T.K = K; T.max_len = max_len; T.k_E = 0; T.status = 0;
            T.min_kept_exp = K ? (cache->kept[K - 1] & kEmax) : kEmax + 1;
        }
        s_ok = ok;
        ws->spec = ok; ws->spec_ok = 0;
    }
    __syncthreads();
    if (s_ok) {
        const u32 K = cache->K;
        uint8_t* symlen_of_bucket = EB == 8 ? T.symlen_of_bucket : ext->symlen_of_bucket;
        for (u32 b = lane; b < kBuckets; b += kW) {
            const u32 sy = s_sym[b] == 0xFF ? K : s_sym[b];
            symlen_of_bucket[b] = (uint8_t)(sy | (s_len[sy] << 4));
        }
    }
}

// ----------------------------------------------------------------------------- sweeps by wavefronts
// The single sweep of lc_encode_cached, which counts and codes (only counts where the cache holds no usable table): one wavefront per
// chunk, no communication between wavefronts.  Coding, each lane codes its 256 elements into a bit string of its own,
// written word by word to the chunk's slot in the scratch area (lane-private, word k of lane l at slot[32 + 64 k + l]); the
// 64 bit lengths go to the head of the slot, their sum to chunk_bits[c].  Where the strings end up in the blob is decided
// afterwards by k_place, which knows all sizes.  A full chunk takes the fast path, off alignment too (2^25 fp32 laplace elements
// off alignment 150 us the call by element loads, 95 so, as aligned; bf16 200 -> 89): rows are fetched eight
// at a time, one batch ahead (and the next chunk's first batch before the current one ends), the table look-ups of 16
// elements are issued together and two symbols are coded per look-up.  A ragged chunk takes a plain path.  The
// mantissa extremes of the kept buckets (Section 3.1.1: the representative is the mean of the bucket's largest and smallest
// member) are tracked on the way.
constexpr int kMmCopies = 32;       // LDS copies of the per-symbol extremes, one per lane of a half wave

constexpr u32 kStageRows = 32;      // code words per lane that a chunk gathers in LDS before they go to its slot

constexpr int kSpecCopies = 2;      // LDS copies of the bucket histogram in the speculative sweep (4 copies leave room for 6
                                    // wavefronts per compute unit instead of 8: 0.443 against 0.428 ms per 2^28 elements)

// Where copy `copy` of bucket b's count lies in PackLds::hist.  The two signs of an exponent would otherwise share an LDS
// bank (512 words apart), and a delta's sign is a coin toss: bit 4 of the index is flipped for the negative half.
__device__ __forceinline__ u32 hist_slot(u32 b, u32 copy) { return (b * kSpecCopies + copy) ^ ((b >> 8) << 4); }

struct PackLds {
    uint8_t sym8[512];               // bucket -> symbol << 3
    u32 codelen[kMaxSym];            // (code << 5) | len
    uint2 pair[256];                 // (symbol a, symbol b) -> {code of a followed by b, its length}
    u32 mn[kMaxSym * kMmCopies], mx[kMaxSym * kMmCopies];   // extremes of the delta bit patterns per symbol
    alignas(16) u32 stage[kStageRows * kW];                 // word k of lane l at [64 k + l], as in the slot
    u32 hist[512 * kSpecCopies];                            // bucket populations
};

// chunk_bits[c] = payload bits of chunk c; group_words[g] = record words of chunks 64g .. 64g+63
// (integer atomics: the sums do not depend on the order of arrival).
// One chunk's work as the coding loop sees it: the vector it belongs to, its index there, and where its
// code words, its bit count and its group's word sum go.
struct ChunkRef {
    const void* w; const void* w_ref;
    u64 n;
    u32 c;
    u32* slot; u32* bits_at; u32* group_at;
    bool valid, fast;            // fast: a full chunk
    bool by_parts;               // a chunk that is mostly merged: coded part by part, and
    u32 parts;                   // which of its whole parts have to be read
};

// In chunk_bits beside a chunk's payload bits (at most 16384 * 15).  kMergedChunk: a full chunk whose largest exponent (sweep
// 1 recorded it) lies below every kept bucket: all 16384 symbols are the merged one (Section 3.1.1, priority promotion) and
// each lane's string is 256 copies of its code.  Such a chunk gets no slot: sweep 2 only notes its size, and k_place writes
// the repeated code straight into the blob.  kRawChunk: the slot holds lane strings that k_place has to join; without it
// the record as it goes into the blob.
constexpr u32 kMergedChunk = 0x80000000u, kRawChunk = 0x40000000u, kChunkBits = 0x3FFFFFFFu;

// Lane strings in the slot: their lengths.
__device__ __forceinline__ void finish_lane_sizes(const ChunkRef& ch, u32 nb, u32 nw) {
    const u32 lane = lane_id();
    const u32 bits = 32 * nw + nb;
    reinterpret_cast<uint16_t*>(ch.slot)[lane] = (uint16_t)bits;
    const u32 total = wave_sum32(bits);
    if (lane == 0) {
        *ch.bits_at = total | kRawChunk;
        atomicAdd(ch.group_at, kLaneBitsWords + ((total + 31) >> 5));
    }
}

// Any size, any alignment, one symbol per look-up.  The vector's ragged last chunk is one wavefront's work from
// start to end, so its memory round trips count: the rows that lie wholly inside the vector are fetched as
// in a full chunk, four at a time and one batch ahead; what is left takes guarded element loads.
constexpr int kPlainRows = 4;

template <bool PACK, int DT>
__device__ __noinline__ void pack_chunk_plain(const ChunkRef ch, PackLds& L) {
    const u32 lane = lane_id();
    const void* __restrict__ w = ch.w; const void* __restrict__ w_ref = ch.w_ref;
    const u64 n = ch.n, base = (u64)ch.c * kChunk;
    u32* slot = ch.slot;
    const u32 mm = lane & (kMmCopies - 1);
    u64 acc = 0;
    u32 nb = 0, nw = 0;
    auto code_row = [&](auto whole, u64 idx, const float (&xa)[4], const float (&xb)[4]) {
        constexpr bool WHOLE = decltype(whole)::value;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            if (WHOLE || idx + v < n) {
                const u32 u = delta_bits(xa[v], xb[v]);
                atomicAdd(&L.hist[hist_slot(u >> 23, lane & (kSpecCopies - 1))], 1u);
                if (!PACK) continue;
                const u32 sy = L.sym8[u >> 23] >> 3;
                const u32 cl = L.codelen[sy];
                atomicMin(&L.mn[sy * kMmCopies + mm], u);
                atomicMax(&L.mx[sy * kMmCopies + mm], u);
                acc = (acc << (cl & 31)) | (cl >> 5);
                nb += cl & 31;
            }
            if (PACK && (v & 1) && nb >= 32) {
                slot[kLaneBitsWords + nw * kW + lane] = (u32)(acc >> (nb - 32));
                ++nw; nb -= 32;
            }
        }
    };
    typedef std::integral_constant<bool, true> yes;
    typedef std::integral_constant<bool, false> no;
    auto row_at_ = [&](u32 r) { return base + (u64)r * kRowElems + lane * kV; };
    // whole rows, in batches of kPlainRows
    u32 r = 0;
    const u64 inside = n > base ? n - base : 0;
    const u32 whole_rows = (u32)min((u64)kR, inside / kRowElems) / kPlainRows * kPlainRows;
    if (whole_rows) {
        float xa[kPlainRows][4], xb[kPlainRows][4], ya[kPlainRows][4], yb[kPlainRows][4];
        auto fetch = [&](float (&a)[kPlainRows][4], float (&b)[kPlainRows][4], u32 r0) {
#pragma unroll
            for (int k = 0; k < kPlainRows; ++k) { load_row_any<DT>(w, row_at_(r0 + k), a[k]); load_row_any<DT>(w_ref, row_at_(r0 + k), b[k]); }
        };
        auto code = [&](const float (&a)[kPlainRows][4], const float (&b)[kPlainRows][4], u32 r0) {
#pragma unroll
            for (int k = 0; k < kPlainRows; ++k) code_row(yes(), row_at_(r0 + k), a[k], b[k]);
        };
        fetch(xa, xb, 0);
        for (; r < whole_rows; r += 2 * kPlainRows) {
            // the batch after this one, or (none left) this one again: loads on every path, see k_hist
            fetch(ya, yb, r + kPlainRows < whole_rows ? r + kPlainRows : r);
            code(xa, xb, r);
            if (r + kPlainRows >= whole_rows) { r += kPlainRows; break; }
            fetch(xa, xb, r + 2 * kPlainRows < whole_rows ? r + 2 * kPlainRows : r);
            code(ya, yb, r + kPlainRows);
        }
    }
    for (; r < kR && base + (u64)r * kRowElems < n; r += kPlainRows) {
        float xa[kPlainRows][4], xb[kPlainRows][4];
#pragma unroll
        for (int k = 0; k < kPlainRows; ++k) { load_row<false, DT>(w, row_at_(r + k), n, xa[k]); load_row<false, DT>(w_ref, row_at_(r + k), n, xb[k]); }
#pragma unroll
        for (int k = 0; k < kPlainRows; ++k) code_row(no(), row_at_(r + k), xa[k], xb[k]);
    }
    if (!PACK) return;
    if (nb > 0) slot[kLaneBitsWords + nw * kW + lane] = (u32)(acc << (32 - nb));
    finish_lane_sizes(ch, nb, nw);
}

// element index of this lane's 4 elements in row r of chunk c
__device__ __forceinline__ u64 row_at(u32 c, u32 r) { return (u64)c * kChunk + (u64)(r * kW + lane_id()) * kV; }

constexpr int kPackPF = 8;          // rows per prefetch batch of the coding loop

// `rot`: the row a wavefront starts a chunk with (a multiple of kPackPF; rows wrap around).  Coding has to take the
// rows in order (0); counting does not, and wavefronts that start their chunks together on the same row keep asking the
// same few memory channels at a time: chunk starts are 64 KiB apart, and a bare read of two arrays in this pattern runs
// at 5.9 TB/s, with every wavefront starting one batch of rows later than its neighbour at 6.8.
template <int DT>
__device__ __forceinline__ void fetch_first_batch(const ChunkRef& ch, typename Raw<DT>::type (&A)[kPackPF],
                                                  typename Raw<DT>::type (&B)[kPackPF], u32 rot = 0) {
#pragma unroll
    for (int k = 0; k < kPackPF; ++k) { A[k] = load_raw_any<DT>(ch.w, row_at(ch.c, rot + k)); B[k] = load_raw_any<DT>(ch.w_ref, row_at(ch.c, rot + k)); }
}

// A full chunk whose first batch of rows is already in A0/B0; leaves the first batch of `next`
// there if that chunk takes this path too.
template <bool ROWCHK, bool PACK, int DT>
__device__ __forceinline__ void pack_chunk_fast(const ChunkRef& cur, const ChunkRef& next,
                                                typename Raw<DT>::type (&A0)[kPackPF], typename Raw<DT>::type (&B0)[kPackPF],
                                                u32 K8, PackLds& L, u32 rot = 0) {
    constexpr int PF = kPackPF;
    static_assert((kR & (kR - 1)) == 0 && kR % (2 * kPackPF) == 0, "rows wrap with a mask");
    typedef typename Raw<DT>::type raw_t;
    const u32 lane = lane_id();
    const u32 mm = lane & (kMmCopies - 1);
    const void* __restrict__ w = cur.w; const void* __restrict__ w_ref = cur.w_ref;
    const u32 c = cur.c;
    raw_t A1[PF], B1[PF];
    const bool next_fast = next.valid && next.fast;
    u32* lane_words = cur.slot + kLaneBitsWords + lane;
    u64 acc = 0;
    u32 nb = 0, nw = 0;                       // bits waiting in acc, words written
    // Lanes fill their words at different times; gathering them in LDS and storing whole rows at
    // the end of the chunk turns many partial-line stores into a few full ones.
    auto flush = [&]() {
        if (nb >= 32) {
            const u32 word = (u32)(acc >> (nb - 32));
            if (nw < kStageRows) L.stage[nw * kW + lane] = word;
            else lane_words[nw * kW] = word;
            ++nw; nb -= 32;
        }
    };
    // Four rows at a time: all table look-ups of the 16 elements are issued together, so the
    // LDS latency is paid twice per group instead of three times per row; only the shift/or
    // chain that grows the lane's bit string is serial.
    auto group = [&](const raw_t* a, const raw_t* b) {
        u32 u[16], t[16];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            float xa[4], xb[4];
            unpack<DT>(a[k], xa); unpack<DT>(b[k], xb);
#pragma unroll
            for (int v = 0; v < 4; ++v) u[4 * k + v] = delta_bits(xa[v], xb[v]);
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) atomicAdd(&L.hist[hist_slot(u[i] >> 23, lane & (kSpecCopies - 1))], 1u);
        if (!PACK) return;
#pragma unroll
        for (int i = 0; i < 16; ++i) t[i] = L.sym8[u[i] >> 23];
        uint2 p[8];
#pragma unroll
        for (int i = 0; i < 8; ++i)
            p[i] = *reinterpret_cast<const uint2*>(reinterpret_cast<const uint8_t*>(L.pair) + ((t[2 * i] << 4) | t[2 * i + 1]));
        u32 tmin = t[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) tmin = min(tmin, t[i]);
        if (__any(tmin < K8)) {
            // some lane holds a kept element: everyone updates the extremes of its symbols
            // (the merged symbol has a slot of its own that nobody reads)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                atomicMin(&L.mn[t[i] * (kMmCopies / 8) + mm], u[i]);
                atomicMax(&L.mx[t[i] * (kMmCopies / 8) + mm], u[i]);
            }
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            acc = (acc << p[i].y) | p[i].x; nb += p[i].y;
            if (!ROWCHK || (i & 1)) flush();
        }
    };
    // (row: the chunk's row that step r0 starts with; rot is 0 unless this is the counting sweep)
    auto row = [&](u32 r) { return !PACK ? ((r + rot) & (kR - 1)) : r; };
    for (u32 r0 = 0; r0 < kR; r0 += 2 * PF) {
#pragma unroll
        for (int k = 0; k < PF; ++k) { A1[k] = load_raw_any<DT>(w, row_at(c, row(r0 + PF) + k)); B1[k] = load_raw_any<DT>(w_ref, row_at(c, row(r0 + PF) + k)); }
        group(A0, B0); group(A0 + 4, B0 + 4);
        if (r0 + 2 * PF < kR) {
#pragma unroll
            for (int k = 0; k < PF; ++k) { A0[k] = load_raw_any<DT>(w, row_at(c, row(r0 + 2 * PF) + k)); B0[k] = load_raw_any<DT>(w_ref, row_at(c, row(r0 + 2 * PF) + k)); }
        } else if (next_fast) {
            fetch_first_batch<DT>(next, A0, B0, !PACK ? rot : 0u);
        }
        group(A1, B1); group(A1 + 4, B1 + 4);
    }
    if (!PACK) return;
    // the last, partly filled word, then rows 0 .. (most words of any lane) - 1, four rows per store
    if (nb > 0) {
        const u32 word = (u32)(acc << (32 - nb));
        if (nw < kStageRows) L.stage[nw * kW + lane] = word;
        else lane_words[nw * kW] = word;
    }
    u32 rows = min(nw + (nb > 0 ? 1u : 0u), kStageRows);
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) rows = max(rows, (u32)__shfl_xor(rows, d, 64));
    {
        const uint4* src = reinterpret_cast<const uint4*>(L.stage);
        uint4* dst = reinterpret_cast<uint4*>(cur.slot + kLaneBitsWords);
        for (u32 i = lane; i < rows * (kW / 4); i += kW) dst[i] = src[i];
    }
    finish_lane_sizes(cur, nb, nw);
}

// The loop of one wavefront over the chunks its source hands out.  Src::take() is the wavefront's next chunk,
// Src::K8() is symbol K << 3 of the table.
// ROWSEL: 1 = a lane's 64-bit accumulator can take a whole row (31 waiting bits + 4 codes of <= 8 bits) between flushes.
template <bool PACK, int DT, int ROWSEL, typename Src>
__device__ __forceinline__ void pack_loop(Src& src, PackLds& L) {
    typedef typename Raw<DT>::type raw_t;
    raw_t A0[kPackPF], B0[kPackPF];
    // the counting sweep: every wavefront starts its chunks one batch of rows after its neighbour (see fetch_first_batch)
    const u32 rot = !PACK ? (blockIdx.x % (kR / kPackPF)) * kPackPF : 0u;
    // (behind a chunk that was not coded from these arrays nothing in them lives on: without a word about that the compiler
    // kept their registers through the calls to the other paths, 256 in all for kb_pack, one wavefront per SIMD)
    auto forget = [&]() {
#pragma unroll
        for (int k = 0; k < kPackPF; ++k) { A0[k] = raw_t{}; B0[k] = raw_t{}; }
    };
    ChunkRef cur = src.take();
    if (cur.valid && cur.fast) fetch_first_batch<DT>(cur, A0, B0, rot);
    while (cur.valid) {
        const ChunkRef next = src.take();
        if constexpr (!PACK) {
            // counting only
            if (!cur.fast) {
                pack_chunk_plain<PACK, DT>(cur, L);
                forget();
                if (next.valid && next.fast) fetch_first_batch<DT>(next, A0, B0, rot);
            } else {
                pack_chunk_fast<true, PACK, DT>(cur, next, A0, B0, src.K8(), L, rot);
            }
        } else if (!cur.fast) {
            pack_chunk_plain<PACK, DT>(cur, L);
            forget();
            if (next.valid && next.fast) fetch_first_batch<DT>(next, A0, B0);
        } else if (ROWSEL == 1) {
            pack_chunk_fast<true, PACK, DT>(cur, next, A0, B0, src.K8(), L);
        } else {
            pack_chunk_fast<false, PACK, DT>(cur, next, A0, B0, src.K8(), L);
        }
        cur = next;
    }
}

// Binary64 parameters: which of the first `whole` parts of a chunk (32 of 512 elements, two bytes per recorded maximum, 11
// exponent bits) hold an exponent of a kept bucket; false if those are more than a quarter of a chunk's parts (the chunk
// then takes the usual path).
__device__ __forceinline__ bool parts_to_read64(const uint16_t* maxima, u32 min_kept_exp, u32 whole, u32* parts) {
    const u32* p = reinterpret_cast<const u32*>(maxima);
    u32 mask = 0;
    for (u32 i = 0; i < 16; ++i) {
        const u32 word = load_uniform(p + i);
        mask |= ((word & 0xFFFFu) >= min_kept_exp ? 1u : 0u) << (2 * i);
        mask |= ((word >> 16) >= min_kept_exp ? 1u : 0u) << (2 * i + 1);
    }
    if (whole < 32) mask &= (1u << whole) - 1u;
    *parts = mask;
    return (u32)__popc(mask) <= 8u;
}

// The chunks of one vector that have to be read, dealt round-robin to the wavefronts of the grid: all of
// them, or with chunk_list the `listed` ones named there.
struct VectorChunks {
    const void* w; const void* w_ref;
    u64 n;
    u32* prov; u32 slot_words; u32* chunk_bits; u32* group_words;
    u32 nchunks;
    u32 k8; bool row;
    const u32* chunk_list; u32 listed;
    u32 pos;
    const uint8_t* batch_max; u32 parts_per_chunk, min_kept_exp, cl_merged;     // binary64: what sweep 1 recorded per 4 KiB batch, or null
    __device__ __forceinline__ u32 merged_codelen() const { return cl_merged; }
    __device__ __forceinline__ ChunkRef ref(u32 c, bool valid) const {
        ChunkRef ch;
        ch.c = c;
        ch.valid = valid;
        ch.w = w; ch.w_ref = w_ref; ch.n = n;
        ch.fast = (u64)(c + 1) * kChunk <= n;
        ch.slot = prov + (u64)c * slot_words;
        ch.bits_at = chunk_bits + c;
        ch.group_at = group_words + (c >> 6);
        ch.parts = 0; ch.by_parts = false;
        if (valid && batch_max) {
            const u64 inside = n - (u64)c * kChunk, part_elems = kChunk / parts_per_chunk;
            const u32 whole = inside >= kChunk ? parts_per_chunk : (u32)(inside / part_elems);
            // (less than one whole part: the guarded path)
            ch.by_parts = whole != 0 && parts_to_read64(reinterpret_cast<const uint16_t*>(batch_max) + (u64)c * parts_per_chunk, min_kept_exp, whole, &ch.parts);
        }
        return ch;
    }
    __device__ __forceinline__ ChunkRef take() {
        const u32 i = blockIdx.x + (pos++) * gridDim.x;
        if (!chunk_list) return ref(i, i < nchunks);
        return i < listed ? ref(load_uniform(chunk_list + i), true) : ref(nchunks, false);
    }
    __device__ __forceinline__ u32 K8() const { return k8; }
};

__device__ __forceinline__ void pack_setup(PackLds& L, const Table& T, u32 lane) {
    for (u32 i = lane; i < 512; i += 64) L.sym8[i] = (uint8_t)((T.symlen_of_bucket[i] & 15) << 3);
    if (lane < kMaxSym) L.codelen[lane] = T.codelen[lane];
    for (u32 i = lane; i < 256; i += 64) {
        const u32 ca = T.codelen[i >> 4], cb = T.codelen[i & 15];
        L.pair[i] = make_uint2(((ca >> 5) << (cb & 31)) | (cb >> 5), (ca & 31) + (cb & 31));
    }
    for (u32 i = lane; i < kMaxSym * kMmCopies; i += 64) { L.mn[i] = 0xFFFFFFFFu; L.mx[i] = 0; }
}

__device__ __forceinline__ void pack_merge_extremes(PackLds& L, EncState* ws, u32 K, u32 lane) {
    if (lane < K) {
        u32 mn = 0xFFFFFFFFu, mx = 0;
#pragma unroll
        for (int k = 0; k < kMmCopies; ++k) { mn = min(mn, L.mn[lane * kMmCopies + k]); mx = max(mx, L.mx[lane * kMmCopies + k]); }
        // Wavefronts that code chunks of one vector finish at about the same time, and atomics on one cache line are
        // served one after the other (a 1000-chunk tensor's queued up for 30 us): each workgroup hands its extremes to
        // one of kExtCopies copies, which the workgroup that writes the header joins.
        const u32 copy = blockIdx.x % kExtCopies;
        if (mn <= mx) { atomicMin(&ws->mmin[copy][lane], mn & 0x7FFFFFu); atomicMax(&ws->mmax[copy][lane], mx & 0x7FFFFFu); }
    }
}

// The chunks k_table left off the list (full ones that hold merged elements only): their sizes, a group of 64 per step.
__device__ __forceinline__ void note_merged_chunks(const Table& T, u64 n, u32* chunk_bits, u32* group_words,
                                                   const u32* chunk_maxexp) {
    const u32 lane = lane_id();
    const u32 nfull = (u32)(n / kChunk), min_kept_exp = T.min_kept_exp, len_merged = T.codelen[T.K] & 31;
    for (u32 c0 = (blockIdx.x * blockDim.x + threadIdx.x) & ~(kW - 1); c0 < nfull; c0 += gridDim.x * blockDim.x) {
        const u32 c = c0 + lane;
        const bool merged = c < nfull && chunk_maxexp[maxexp_slot(c)] < min_kept_exp;
        if (merged) chunk_bits[c] = kMergedChunk | (kChunk * len_merged);
        const u32 count = (u32)__popcll(__ballot(merged));
        if (lane == 0 && count) atomicAdd(&group_words[c0 >> 6], count * (kLaneBitsWords + kChunk / 32 * len_merged));
    }
}

// ----------------------------------------------------------------------------- coding by workgroups
// Sweep 2 (fp32, bf16, fp16, and from staged keys): a workgroup of eight wavefronts per chunk, wavefront v coding rows
// 8 v .. 8 v + 7, so that every lane's string of 256 codes grows in eight parts of 32 side by side.  A workgroup codes one
// chunk and ends: its rows are asked for as soon as it is known that they have to be read, and what overlaps one chunk's waits with
// another's work is that several workgroups share a compute unit.  The parts (up to kPartWords words of every lane) stay in
// LDS; once all lengths are known, each thread ORs its part, shifted, into the chunk's payload there, and lane lengths and
// payload go to the chunk's slot as the record that the blob will hold: k_place then only copies it.  A chunk whose
// strings outgrow these areas (a layer above the others' scale, say: symbols that are rare in the vector as a whole) is
// coded again, straight to its places in the payload (finish_long).
// Before, a wavefront walked over chunks with its next rows in flight (2 wavefronts per SIMD, or 1, by its registers);
// k_pack and k_place, before -> after: 2^20 fp32 elements 19.3 + 4.8 -> 7.6 + 3.6 us, 2^27 bf16 138 + 27 -> 119 + 19 us,
// 2^28 fp32 430 + 45 -> 426 + 33 us, from keys 139 + 45 -> 114 + 33 us; 161 tensors of 25.6 M (kb_list, kb_pack, kb_place)
// 5 + 44 + 12 -> 0 + 45 + 7 us.
// (Workgroups that stay and walk over chunks, the next one's rows in flight: 159 us on the bf16 vector.)
constexpr u32 kWgWaves = 8, kWgRows = kR / kWgWaves, kWgThreads = kWgWaves * kW;
constexpr u32 kPartWords = 7;           // words of a lane's part: 32 codes of 7 bits
constexpr u32 kPayloadWords = 2560;     // words of a chunk's payload: 5 bits per element

constexpr u32 kPairs = kMaxSym + 1;

struct PackWg {
    uint8_t sym8[512];                   // bucket -> symbol << 3
    u32 codelen[kMaxSym];                // (code << 5) | len
    uint2 pair[kPairs * kPairs];         // (symbol a, symbol b) -> {code of a followed by b, its length}; symbol 16: none, no bits
    u32 mn[kMaxSym * kMmCopies], mx[kMaxSym * kMmCopies];      // extremes of the delta bit patterns per symbol
    u32 bits[kWgWaves][kW];              // lengths of the parts
    alignas(16) u32 part[kWgWaves][kPartWords * kW]; // word k of lane l at [64 k + l]
    alignas(16) u32 payload[kPayloadWords];
    u32 overflow;                        // some part does not fit its area
};

// A lane's part while it grows.
struct LanePart {
    u32 acc, nb;                         // the last nb < 32 bits of acc wait (what stands above them is of no account)
    u32 *words, *first;                  // where the next word goes in this lane's column of PackWg::part, and the first one
    __device__ __forceinline__ void start(PackWg& L, u32 v) { acc = 0; nb = 0; words = first = L.part[v] + lane_id(); }
    __device__ __forceinline__ void put(u32 word) { if (words < first + kPartWords * kW) *words = word; words += kW; }
    // len <= 31; what stands above `code` is zero
    __device__ __forceinline__ void append(u32 code, u32 len) {
        const u32 before = acc, had = nb;
        acc = (acc << len) | code; nb += len;
        if (nb >= 32) { put(__builtin_amdgcn_alignbit(before, code << (32 - len), had)); nb -= 32; }
    }
    __device__ __forceinline__ u32 bits() const { return 32 * ((u32)(words - first) / kW) + nb; }
};

// Two rows, their symbols (<< 3) looked up: only the chain that grows the lane's part is serial.  Four codes are put together
// first, as long as they take at most 31 bits in every lane (codes of up to 7 bits always do), and join the part at once.
__device__ __forceinline__ void code_symbols(const u32 (&t)[8], PackWg& L, LanePart& S) {
    uint2 p[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) p[i] = *reinterpret_cast<const uint2*>(reinterpret_cast<const uint8_t*>(L.pair) + (t[2 * i] * kPairs + t[2 * i + 1]));
    const u32 len0 = p[0].y + p[1].y, len1 = p[2].y + p[3].y;
    if (__any(max(len0, len1) > 31)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) S.append(p[i].x, p[i].y);
    } else {
        S.append((p[0].x << p[1].y) | p[1].x, len0);
        S.append((p[2].x << p[3].y) | p[3].x, len1);
    }
}

// Two rows' deltas: the look-ups of the 8 elements are issued together.
__device__ __forceinline__ void code_deltas(const u32* u, u32 K8, PackWg& L, LanePart& S) {
    u32 t[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) t[i] = L.sym8[u[i] >> 23];
    u32 tmin = t[0];
#pragma unroll
    for (int i = 1; i < 8; ++i) tmin = min(tmin, t[i]);
    if (__any(tmin < K8)) {              // (the merged symbol has a slot of its own that nobody reads)
        const u32 copy = lane_id() & (kMmCopies - 1);
#pragma unroll
        for (int i = 0; i < 8; ++i) { atomicMin(&L.mn[t[i] * (kMmCopies / 8) + copy], u[i]); atomicMax(&L.mx[t[i] * (kMmCopies / 8) + copy], u[i]); }
    }
    code_symbols(t, L, S);
}

// Two rows of w and w_ref.
template <int DT>
__device__ __forceinline__ void code_rows2(const typename Raw<DT>::type* a, const typename Raw<DT>::type* b, u32 K8, PackWg& L, LanePart& S) {
    u32 u[8];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        float xa[4], xb[4];
        unpack<DT>(a[k], xa); unpack<DT>(b[k], xb);
#pragma unroll
        for (int v = 0; v < 4; ++v) u[4 * k + v] = delta_bits(xa[v], xb[v]);
    }
    code_deltas(u, K8, L, S);
}

// The first `count` words of the payload to memory, in 16-byte vectors that are aligned to words only.
__device__ __forceinline__ void copy_payload(u32* to, u32 count, const PackWg& L) {
    typedef u32x4 __attribute__((aligned(4))) u32x4_word;
    const u32 nvec = count / 4;
    for (u32 i = threadIdx.x; i < nvec; i += kWgThreads) reinterpret_cast<u32x4_word*>(to)[i] = reinterpret_cast<const u32x4*>(L.payload)[i];
    if (threadIdx.x < (count & 3)) to[4 * nvec + threadIdx.x] = L.payload[4 * nvec + threadIdx.x];
}

// The symbols of a lane's part, 4 bits each, the first in the low bits of s[0]; count of them.
struct PartSymbols { u64 s[2]; u32 count; };

// A chunk whose strings outgrow the workgroup's areas, all wavefronts side by side: where each part goes is known (o: its first
// bit in the payload), so the parts are coded again straight to their places, in as many turns as windows of kPayloadWords
// words hold the payload (3 at most).  Contains barriers; L.payload is cleared when it is called.
// By one wavefront instead, a row at a time: 2^24 fp32 elements of 10 layers at 4 bits 143 us the call, 101 so.
__device__ __forceinline__ void finish_long(u32* payload, const PartSymbols& P, u32 o, u32 nwords, PackWg& L) {
    const u32 t = threadIdx.x;
#pragma unroll 1
    for (u32 base = 0; base < nwords; base += kPayloadWords) {
        if (base != 0) {
            for (u32 i = t; i < kPayloadWords; i += kWgThreads) L.payload[i] = 0;
            __syncthreads();
        }
        u64 acc = 0;
        u32 nb = o & 31, at = (o >> 5) - base;                 // (words before the window wrap to large numbers)
        auto put = [&](u32 word) { if (at < kPayloadWords) atomicOr(&L.payload[at], word); ++at; };
        auto append = [&](u32 code, u32 len) {
            acc = (acc << len) | code; nb += len;
            if (nb >= 32) { put((u32)(acc >> (nb - 32))); nb -= 32; }
        };
        u64 s = P.s[0];
        u32 i = 0;
#pragma unroll 1
        for (; i + 8 <= P.count; i += 8) {                     // two symbols per look-up, four look-ups in flight
            uint2 p[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) { p[k] = L.pair[((u32)s & 15u) * kPairs + ((u32)(s >> 4) & 15u)]; s >>= 8; }
#pragma unroll
            for (int k = 0; k < 4; ++k) append(p[k].x, p[k].y);
            if (i == 8) s = P.s[1];
        }
        if (i == 16) s = P.s[1];
#pragma unroll 1
        for (; i < P.count; ++i) {
            const u32 cl = L.codelen[(u32)s & 15u];
            append(cl >> 5, cl & 31);
            s = i == 15 ? P.s[1] : s >> 4;
        }
        if (nb > 0) put((u32)(acc << (32 - nb)));
        __syncthreads();
        copy_payload(payload + base, min(nwords - base, kPayloadWords), L);
        __syncthreads();
    }
}

// Where the strings of a chunk go, once all parts are coded: known to every thread after part_places (which contains a barrier).
struct PartPlaces {
    u32 mine, o;             // this lane's part: its bits, and its first bit in the payload
    u32 bits;                // the lane's whole string
    u32 total, nwords;       // the chunk's payload in bits and in words
    bool overflow;           // it does not fit the workgroup's areas
};
__device__ __forceinline__ PartPlaces part_places(LanePart& S, u32 v, PackWg& L) {
    const u32 lane = lane_id();
    PartPlaces P;
    P.mine = S.bits();
    if (S.nb > 0) S.put(S.acc << (32 - S.nb));
    L.bits[v][lane] = P.mine;
    if (P.mine > 32 * kPartWords) L.overflow = 1;
    __syncthreads();
    u32 before = 0;
    P.bits = 0;
#pragma unroll
    for (u32 k = 0; k < kWgWaves; ++k) {
        const u32 b = L.bits[k][lane];
        before += k < v ? b : 0u;
        P.bits += b;
    }
    const u32 incl = wave_incl_scan(P.bits);
    P.total = read_lane(incl, kW - 1);
    P.nwords = (P.total + 31) >> 5;
    P.o = incl - P.bits + before;
    P.overflow = L.overflow != 0 || P.nwords > kPayloadWords;
    return P;
}

// The parts joined into the payload (cleared before); the caller's barrier follows.
__device__ __forceinline__ void join_parts(const PartPlaces& P, u32 v, PackWg& L) {
    const u32 sh = P.o & 31, W0 = P.o >> 5, have = (P.mine + 31) >> 5;
    const u32 touched = P.mine ? ((P.o + P.mine - 1) >> 5) - W0 + 1 : 0;
    u32 prev = 0;                                          // (a part of 7 words touches 8 of the payload)
#pragma unroll
    for (u32 j = 0; j <= kPartWords; ++j) {
        const u32 w = j < have && j < kPartWords ? L.part[v][j * kW + lane_id()] : 0;
        if (j < touched) atomicOr(&L.payload[W0 + j], __builtin_amdgcn_alignbit(prev, w, sh));
        prev = w;
    }
}

// All parts are coded: their lengths, the payload, the record.  again(): the symbols of this lane's part once more, for a chunk
// that does not fit its areas.  Contains barriers.
template <typename Again>
__device__ __forceinline__ void finish_parts(const ChunkRef& ch, LanePart& S, u32 v, PackWg& L, const Again& again) {
    const u32 t = threadIdx.x, lane = lane_id();
    const PartPlaces P = part_places(S, v, L);
    const u32 nwords = P.nwords;
    if (v == 0) {
        reinterpret_cast<uint16_t*>(ch.slot)[lane] = (uint16_t)P.bits;
        if (lane == 0) { *ch.bits_at = P.total; atomicAdd(ch.group_at, kLaneBitsWords + nwords); }
    }
    if (P.overflow) { finish_long(ch.slot + kLaneBitsWords, again(), P.o, nwords, L); return; }
    join_parts(P, v, L);
    __syncthreads();
    // the payload in whole vectors (what lies behind its end in the slot nobody reads)
    const u32x4* from = reinterpret_cast<const u32x4*>(L.payload);
    u32x4* to = reinterpret_cast<u32x4*>(ch.slot + kLaneBitsWords);
    for (u32 i = t; i < (nwords + 3) / 4; i += kWgThreads) to[i] = from[i];
}

// 4 elements from index i on, those at n and behind read as zero; any alignment
template <int DT>
__device__ __forceinline__ typename Raw<DT>::type load_raw_guarded(const void* base, u64 i, u64 n) {
    if constexpr (DT == kF32) {
        const float* p = static_cast<const float*>(base) + i;
        float x[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = i + e < n ? p[e] : 0.0f;
        return make_float4(x[0], x[1], x[2], x[3]);
    } else {
        const uint16_t* p = static_cast<const uint16_t*>(base) + i;
        u32 x[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = i + e < n ? p[e] : 0u;
        return make_uint2(x[0] | (x[1] << 16), x[2] | (x[3] << 16));
    }
}

__device__ __forceinline__ void pair_setup(PackWg& L, const u32* codelen) {
    const u32 t = threadIdx.x, a = t / kPairs, b = t % kPairs;
    if (t >= kPairs * kPairs) return;
    const u32 ca = a < kMaxSym ? codelen[a] : 0u, cb = b < kMaxSym ? codelen[b] : 0u;
    L.pair[t] = make_uint2(((ca >> 5) << (cb & 31)) | (cb >> 5), (ca & 31) + (cb & 31));
}

// The workgroup's tables, extremes and areas; a barrier of the caller's follows.  (kWgThreads = 512 buckets)
__device__ __forceinline__ void pack_setup(PackWg& L, const Table& T) {
    const u32 t = threadIdx.x;
    const u32 sl = T.symlen_of_bucket[t];
    const u32 own = t < kMaxSym ? T.codelen[t] : 0u;
    pair_setup(L, T.codelen);
    L.sym8[t] = (uint8_t)((sl & 15) << 3);
    if (t < kMaxSym) L.codelen[t] = own;
    static_assert(kWgThreads == 512 && kMaxSym * kMmCopies == 512, "one entry per thread");
    L.mn[t] = 0xFFFFFFFFu; L.mx[t] = 0;
    if (t == 0) L.overflow = 0;
    for (u32 i = t; i < kPayloadWords; i += kWgThreads) L.payload[i] = 0;
}

// A full chunk whose largest exponent `maxexp` lies below every kept bucket holds the merged symbol only: it gets its size
// and no slot (as in note_merged_chunks).  Returns whether it is one, the same in every thread.
__device__ __forceinline__ bool noted_as_merged(const ChunkRef& ch, const Table& T, u32 maxexp) {
    if ((u64)(ch.c + 1) * kChunk > ch.n || maxexp >= T.min_kept_exp) return false;
    if (threadIdx.x == 0) {
        const u32 len_merged = T.codelen[T.K] & 31;
        *ch.bits_at = kMergedChunk | (kChunk * len_merged);
        atomicAdd(ch.group_at, kLaneBitsWords + kChunk / 32 * len_merged);
    }
    return true;
}

// What sweep 1 recorded of the parts this wavefront's rows lie in: the largest exponent of each 4 KiB part of a chunk, one byte
// each from `parts` on (16 parts of 4-byte elements, 8 of 2-byte).  Asked for together with the chunk's own maximum.
constexpr u32 kReadAllParts = 0xFFFFFFFFu;
template <int DT>
__device__ __forceinline__ u32 part_word(const uint8_t* parts) {
    const u32 v = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    return load_uniform(reinterpret_cast<const u32*>(parts) + (elem_bytes<DT>() == 4 ? v / 2 : v / 4));
}

// Codes the chunk with table T (in memory).  maxima: part_word of the chunk, or kReadAllParts; parts of a full chunk
// below every kept bucket are not read.  A full chunk takes vector loads at any alignment, in one wait; by guarded loads of single
// elements, off alignment, fp32 2^25 laplace elements 146 us the call and 120 so, 2^24 94 and 78, bf16 2^26 225 and 155, 32 layers
// of 2^20 in a batch fp32 202 and 143, bf16 354 and 120 (aligned ones the same to 1 %).
template <int DT>
__device__ __forceinline__ void pack_chunk_wg(const ChunkRef& ch, const Table& T, u32 maxima, EncState* ws, PackWg& L) {
    typedef typename Raw<DT>::type raw_t;
    constexpr u32 kPartRows = 4096 / (kRowElems * elem_bytes<DT>()), H = kWgRows / 2;      // 4 or 8 rows per part
    const u32 lane = lane_id(), v = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), first_row = kWgRows * v;
    raw_t A[kWgRows], B[kWgRows];
    bool skip[2] = {false, false};           // rows first_row .. + 3, and the 4 behind them: merged elements only
    if (ch.fast) {
#pragma unroll
        for (u32 h = 0; h < 2; ++h) skip[h] = ((maxima >> (8 * ((first_row + H * h) / kPartRows % 4))) & 255u) < T.min_kept_exp;
#pragma unroll
        for (u32 h = 0; h < 2; ++h) {
            if (skip[h]) continue;
#pragma unroll
            for (u32 k = H * h; k < H * h + H; ++k) { A[k] = load_raw_any<DT>(ch.w, row_at(ch.c, first_row + k)); B[k] = load_raw_any<DT>(ch.w_ref, row_at(ch.c, first_row + k)); }
        }
    } else {
#pragma unroll
        for (u32 k = 0; k < kWgRows; ++k) { A[k] = load_raw_guarded<DT>(ch.w, row_at(ch.c, first_row + k), ch.n); B[k] = load_raw_guarded<DT>(ch.w_ref, row_at(ch.c, first_row + k), ch.n); }
    }
    const u32 K8 = T.K << 3;
    pack_setup(L, T);
    __syncthreads();
    LanePart S;
    S.start(L, v);
    if (ch.fast) {
#pragma unroll
        for (u32 h = 0; h < 2; ++h) {
            if (skip[h]) {
                // the merged code 16 times, as many copies per step as fit 31 bits (a chunk with such a part holds merged
                // elements, so their symbol has a code)
                const u32 cl = L.codelen[K8 >> 3], len = cl & 31, per_step = len ? 31 / len : 1;
                u32 run = 0;
#pragma unroll 1
                for (u32 i = 0; i < per_step; ++i) run = (run << len) | (cl >> 5);
#pragma unroll 1
                for (u32 left = H * kV; left != 0;) {
                    const u32 k = left < per_step ? left : per_step;
                    S.append(run >> ((per_step - k) * len), k * len);
                    left -= k;
                }
            } else {
#pragma unroll
                for (u32 k = H * h; k < H * h + H; k += 2) code_rows2<DT>(A + k, B + k, K8, L, S);
            }
        }
    } else {
#pragma unroll
        for (u32 k = 0; k < kWgRows; ++k) {
            const u64 idx = row_at(ch.c, first_row + k);
            float xa[4], xb[4];
            unpack<DT>(A[k], xa); unpack<DT>(B[k], xb);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (idx + e < ch.n) {
                    const u32 u = delta_bits(xa[e], xb[e]), sy8 = L.sym8[u >> 23], cl = L.codelen[sy8 >> 3];
                    const u32 at = sy8 * (kMmCopies / 8) + (lane & (kMmCopies - 1));
                    atomicMin(&L.mn[at], u); atomicMax(&L.mx[at], u);
                    S.append(cl >> 5, cl & 31);
                }
            }
        }
    }
    finish_parts(ch, S, v, L, [&]() {
        PartSymbols P;
        P.count = 0;
#pragma unroll 1
        for (u32 h = 0; h < 2; ++h) {                // (a half at a time, for the registers; behind the first it moves on to s[0])
            raw_t a[H], b[H];
#pragma unroll
            for (u32 k = 0; k < H; ++k) {
                const u64 idx = row_at(ch.c, first_row + H * h + k);
                if (ch.fast) { a[k] = load_raw_any<DT>(ch.w, idx); b[k] = load_raw_any<DT>(ch.w_ref, idx); }
                else { a[k] = load_raw_guarded<DT>(ch.w, idx, ch.n); b[k] = load_raw_guarded<DT>(ch.w_ref, idx, ch.n); }
            }
            u64 s = 0;
#pragma unroll
            for (u32 k = 0; k < H; ++k) {
                const u64 idx = row_at(ch.c, first_row + H * h + k);
                float xa[4], xb[4];
                unpack<DT>(a[k], xa); unpack<DT>(b[k], xb);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    s |= (u64)(L.sym8[delta_bits(xa[e], xb[e]) >> 23] >> 3) << (16 * k + 4 * e);
                    P.count += idx + e < ch.n ? 1u : 0u;      // (those past the vector's end are a lane's last)
                }
            }
            P.s[0] = h == 0 ? s : P.s[0]; P.s[1] = s;
        }
        return P;
    });
    // the extremes: thread t holds copy t mod 32 of symbol t / 32 (see pack_merge_extremes)
    const u32 t = threadIdx.x;
    u32 mn = L.mn[t], mx = L.mx[t];
#pragma unroll
    for (int d = kMmCopies / 2; d >= 1; d >>= 1) { mn = min(mn, (u32)__shfl_xor(mn, d, 64)); mx = max(mx, (u32)__shfl_xor(mx, d, 64)); }
    const u32 sym = t / kMmCopies, copy = blockIdx.x % kExtCopies;
    if (t % kMmCopies == 0 && sym < (K8 >> 3) && mn <= mx) { atomicMin(&ws->mmin[copy][sym], mn & 0x7FFFFFu); atomicMax(&ws->mmax[copy][sym], mx & 0x7FFFFFu); }
}

// Which entry of the list workgroup i takes.  The list holds chunks that are 512 apart side by side, so a run of chunks of the
// same cost (a layer's) comes back every nchunks / 512 entries, in a vector of 2^27 elements every 16: one of the 8 dies that
// workgroups are dealt to in turn would get all of them.  Within each 8 entries the order turns by one every 16.  (300 chunks
// of long codes in 2^27 elements: k_pack_keys 92 -> 68 us.)
__device__ __forceinline__ u32 list_entry(u32 i, u32 count) { return (i | 7u) < count ? (i & ~7u) | ((i + (i >> 4)) & 7u) : i; }

// Sweep 2 of one vector, a workgroup per chunk.  chunk_list: the chunks to read (then workgroups beyond the list leave at
// once, having seen to the sizes of the chunks off it); null: every chunk, and chunk_maxexp (or null) tells those that hold
// merged elements only.
// STAY: workgroups take more than one chunk (behind a speculative sweep: see launch_pack).
template <int DT, bool STAY>
__global__ __launch_bounds__(kWgThreads, DT == kF32 || STAY ? 4 : 8) void k_pack(const void* __restrict__ w, const void* __restrict__ w_ref, u64 n,
                                                     EncState* ws, u32* chunk_bits, u32* group_words, const u32* chunk_maxexp,
                                                     const u32* chunk_list, const uint8_t* batch_max, u32* prov, u32 slot_words, u32 nchunks) {
    __shared__ PackWg L;
    const Table& T = ws->table;
    if (T.status != 0 || ws->spec_ok != 0) return;     // nothing to code, or the speculative sweep already did
    if (chunk_list) note_merged_chunks(T, n, chunk_bits, group_words, chunk_maxexp);
    const u32 count = chunk_list ? ws->list_count : nchunks;
    auto chunk = [&](u32 i) {
        const u32 c = chunk_list ? load_uniform(chunk_list + list_entry(i, count)) : i;
        ChunkRef ch;
        ch.w = w; ch.w_ref = w_ref; ch.n = n; ch.c = c;
        ch.slot = prov + (u64)c * slot_words; ch.bits_at = chunk_bits + c; ch.group_at = group_words + (c >> 6);
        ch.fast = (u64)(c + 1) * kChunk <= n;
        constexpr u32 kParts = kChunk * elem_bytes<DT>() / 4096;
        u32 largest = kReadAllParts, maxima = kReadAllParts;
        if (chunk_maxexp) { largest = load_uniform(chunk_maxexp + maxexp_slot(c)); maxima = part_word<DT>(batch_max + (u64)c * kParts); }
        if (!chunk_list && noted_as_merged(ch, T, largest)) return;
        pack_chunk_wg<DT>(ch, T, maxima, ws, L);
    };
    if constexpr (STAY) {
        for (u32 i = blockIdx.x; i < count; i += gridDim.x) { chunk(i); __syncthreads(); }
    } else {
        if (blockIdx.x < count) chunk(blockIdx.x);
    }
}

// ----------------------------------------------------------------------------- k_pack_keys
// Sweep 2 of an encode with staged keys: as k_pack, coded from the 9-bit keys sweep 1 left (16 exponent bytes + 16 sign bits
// per lane and batch of 4 rows) instead of from w and w_ref: 1.125 bytes per element read instead of 8.  The extremes of
// the kept buckets are sweep 1's business then.  A wavefront's 8 rows are two key loads of each kind per lane; the
// vector's ragged last chunk (whose tail has no keys) is coded from w and w_ref.
constexpr u32 kKeyBatches = kR / 4;                        // batches of 4 rows per chunk

__global__ __launch_bounds__(kWgThreads, 8) void k_pack_keys(const void* __restrict__ w, const void* __restrict__ w_ref, u64 n,
                                                          EncState* ws, u32* chunk_bits, u32* group_words, const u32* chunk_maxexp,
                                                          const u32* chunk_list, KeyPlanes keys, u32* prov, u32 slot_words) {
    __shared__ PackWg L;
    const Table& T = ws->table;
    if (T.status != 0) return;
    note_merged_chunks(T, n, chunk_bits, group_words, chunk_maxexp);
    const u32 count = ws->list_count;
    if (blockIdx.x >= count) return;
    const u32 c = load_uniform(chunk_list + list_entry(blockIdx.x, count));
    ChunkRef ch;
    ch.w = w; ch.w_ref = w_ref; ch.n = n; ch.c = c;
    ch.slot = prov + (u64)c * slot_words; ch.bits_at = chunk_bits + c; ch.group_at = group_words + (c >> 6);
    ch.fast = false;
    if ((u64)(c + 1) * kChunk > n) { pack_chunk_wg<kF32>(ch, T, kReadAllParts, ws, L); return; }
    constexpr u32 kMine = kWgRows / 4;
    const u32 v = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const u64 at = ((u64)c * kKeyBatches + v * kMine) * kW + lane_id();
    u32x4 exps[kMine];
    u32 signs[kMine];
#pragma unroll
    for (u32 b = 0; b < kMine; ++b) {
        exps[b] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(keys.exp) + at + b * kW);
        signs[b] = __builtin_nontemporal_load(keys.sign + at + b * kW);
    }
    pack_setup(L, T);
    __syncthreads();
    LanePart S;
    S.start(L, v);
#pragma unroll
    for (u32 b = 0; b < kMine; ++b) {
        const u32 wv[4] = {exps[b].x, exps[b].y, exps[b].z, exps[b].w};
#pragma unroll
        for (int h = 0; h < 16; h += 8) {
            u32 t[8];
#pragma unroll
            for (int i = 0; i < 8; ++i)             // bucket id = sign << 8 | exponent, as the top 9 bits of the delta
                t[i] = L.sym8[((wv[(h + i) >> 2] >> (8 * (i & 3))) & 255u) | (((signs[b] >> (h + i)) & 1u) << 8)];
            code_symbols(t, L, S);
        }
    }
    finish_parts(ch, S, v, L, [&]() {
        PartSymbols P;
        P.count = kWgRows * kV;
#pragma unroll
        for (u32 b = 0; b < kMine; ++b) {
            const u32x4 x = reinterpret_cast<const u32x4*>(keys.exp)[at + b * kW];
            const u32 sign = keys.sign[at + b * kW], wv[4] = {x.x, x.y, x.z, x.w};
            P.s[b] = 0;
#pragma unroll
            for (int i = 0; i < 16; ++i) P.s[b] |= (u64)(L.sym8[((wv[i >> 2] >> (8 * (i & 3))) & 255u) | (((sign >> i) & 1u) << 8)] >> 3) << (4 * i);
        }
        return P;
    });
}

// ----------------------------------------------------------------------------- k_pack64
// Sweep 2 for binary64 parameters: the same chunks, slots and lane strings; the symbol of an element comes from the
// top 12 bits of its binary64 delta, the extremes are 64-bit patterns.  One symbol per look-up, rows fetched four
// at a time (a row is 32 bytes per lane), code words stored as they fill.
constexpr int kMmCopies64 = 16;

struct PackLds64 {
    uint8_t sym[kBuckets64];
    u32 codelen[kMaxSym];
    unsigned long long mn[kMaxSym * kMmCopies64], mx[kMaxSym * kMmCopies64];
};

template <bool WHOLE>            // WHOLE: a full chunk
__device__ __forceinline__ void pack_chunk64(const ChunkRef& ch, PackLds64& L, u32 K) {
    constexpr int RB = 4;
    const u32 lane = lane_id();
    const u64 n = ch.n, base = (u64)ch.c * kChunk;
    u32* lane_words = ch.slot + kLaneBitsWords + lane;
    const u32 mm = lane & (kMmCopies64 - 1);
    u64 acc = 0;
    u32 nb = 0, nw = 0;
    for (u32 r0 = 0; r0 < kR && (WHOLE || base + (u64)r0 * kRowElems < n); r0 += RB) {
        double xa[RB][4], xb[RB][4];
#pragma unroll
        for (int k = 0; k < RB; ++k) {
            const u64 idx = base + (u64)(r0 + k) * kRowElems + lane * kV;
            if (WHOLE) { load_row_any<kF64>(ch.w, idx, xa[k]); load_row_any<kF64>(ch.w_ref, idx, xb[k]); }
            else { load_row64(ch.w, idx, n, xa[k]); load_row64(ch.w_ref, idx, n, xb[k]); }
        }
#pragma unroll
        for (int k = 0; k < RB; ++k) {
            const u64 idx = base + (u64)(r0 + k) * kRowElems + lane * kV;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                if (WHOLE || idx + v < n) {
                    const u64 u = delta_bits(xa[k][v], xb[k][v]);
                    const u32 sy = L.sym[bucket_of(u)];
                    const u32 cl = L.codelen[sy];
                    if (sy < K) { atomicMin(&L.mn[sy * kMmCopies64 + mm], u); atomicMax(&L.mx[sy * kMmCopies64 + mm], u); }
                    acc = (acc << (cl & 31)) | (cl >> 5);
                    nb += cl & 31;
                }
                if ((v & 1) && nb >= 32) {
                    lane_words[nw * kW] = (u32)(acc >> (nb - 32));
                    ++nw; nb -= 32;
                }
            }
        }
    }
    if (nb > 0) lane_words[nw * kW] = (u32)(acc << (32 - nb));
    finish_lane_sizes(ch, nb, nw);
}

// A chunk of which at most a quarter of the 4 KiB parts (2 rows of doubles each; bit p of `parts` set: part p has to be read)
// hold anything but merged elements: only those are fetched, and the merged code stands for every element of the others.
__device__ __noinline__ void pack_chunk64_parts(const ChunkRef ch, u32 cl_merged, PackLds64& L, u32 K) {
    constexpr u32 kRowsPerPart = 2, kParts = kR / kRowsPerPart;
    const u32 lane = lane_id();
    u32* lane_words = ch.slot + kLaneBitsWords + lane;
    const u32 mm = lane & (kMmCopies64 - 1);
    u64 acc = 0;
    u32 nb = 0, nw = 0;
    auto flush = [&]() {
        if (nb >= 32) { lane_words[nw * kW] = (u32)(acc >> (nb - 32)); ++nw; nb -= 32; }
    };
    const u32 len_merged = cl_merged & 31, per_step = len_merged ? 32 / len_merged : 1;
    u32 run = 0;                                                             // per_step copies of the merged code
    for (u32 i = 0; i < per_step; ++i) run = (run << len_merged) | (cl_merged >> 5);
    auto code_element = [&](double a, double b) {
        const u64 u = delta_bits(a, b);
        const u32 sy = L.sym[bucket_of(u)];
        const u32 cl = L.codelen[sy];
        if (sy < K) { atomicMin(&L.mn[sy * kMmCopies64 + mm], u); atomicMax(&L.mx[sy * kMmCopies64 + mm], u); }
        acc = (acc << (cl & 31)) | (cl >> 5);
        nb += cl & 31;
    };
    const u64 n = ch.n, base = (u64)ch.c * kChunk, inside = n - base;
    const u32 whole = inside >= kChunk ? kParts : (u32)(inside / (kRowsPerPart * kRowElems));
    auto row_idx = [&](u32 r) { return base + (u64)r * kRowElems + lane * kV; };
    for (u32 p = 0; p < whole; ++p) {
        if ((ch.parts >> p) & 1u) {
            double xa[kRowsPerPart][4], xb[kRowsPerPart][4];
#pragma unroll
            for (u32 k = 0; k < kRowsPerPart; ++k) {
                load_row_any<kF64>(ch.w, row_idx(p * kRowsPerPart + k), xa[k]);
                load_row_any<kF64>(ch.w_ref, row_idx(p * kRowsPerPart + k), xb[k]);
            }
#pragma unroll
            for (u32 k = 0; k < kRowsPerPart; ++k) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    code_element(xa[k][v], xb[k][v]);
                    if (v & 1) flush();
                }
            }
        } else {
            for (u32 left = kRowsPerPart * kV; left != 0;) {
                const u32 k = left < per_step ? left : per_step;
                acc = (acc << (k * len_merged)) | (u64)(run >> ((per_step - k) * len_merged));
                nb += k * len_merged;
                flush();
                left -= k;
            }
        }
    }
    if (whole < kParts) {
        // a ragged chunk's last rows (fewer than one part), elements past the end left out
        double xa[kRowsPerPart][4], xb[kRowsPerPart][4];
#pragma unroll
        for (u32 k = 0; k < kRowsPerPart; ++k) {
            load_row64(ch.w, row_idx(whole * kRowsPerPart + k), n, xa[k]);
            load_row64(ch.w_ref, row_idx(whole * kRowsPerPart + k), n, xb[k]);
        }
#pragma unroll
        for (u32 k = 0; k < kRowsPerPart; ++k) {
            const u64 idx = row_idx(whole * kRowsPerPart + k);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                if (idx + v < n) code_element(xa[k][v], xb[k][v]);
                if (v & 1) flush();
            }
        }
    }
    if (nb > 0) lane_words[nw * kW] = (u32)(acc << (32 - nb));
    finish_lane_sizes(ch, nb, nw);
}

__global__ __launch_bounds__(64) void k_pack64(const void* __restrict__ w, const void* __restrict__ w_ref, u64 n,
                                               EncState* ws, Ext64* ext, u32* chunk_bits, u32* group_words,
                                               const u32* chunk_maxexp, const u32* chunk_list, const uint8_t* part_max, u32* prov,
                                               u32 slot_words, u32 nchunks) {
    __shared__ PackLds64 L;
    const u32 lane = threadIdx.x;
    const Table& T = ws->table;
    if (T.status != 0) return;
    const u32 K = T.K;
    for (u32 i = lane; i < kBuckets64; i += kW) L.sym[i] = ext->symlen_of_bucket[i] & 15;
    if (lane < kMaxSym) L.codelen[lane] = T.codelen[lane];
    for (u32 i = lane; i < kMaxSym * kMmCopies64; i += kW) { L.mn[i] = ~0ull; L.mx[i] = 0; }
    __syncthreads();
    VectorChunks src = {w, w_ref, n, prov, slot_words, chunk_bits, group_words, nchunks, K << 3, true,
                        chunk_list, chunk_list ? ws->list_count : 0, 0, chunk_list ? part_max : nullptr, 32u, T.min_kept_exp,
                        T.codelen[K]};
    if (chunk_list) note_merged_chunks(T, n, chunk_bits, group_words, chunk_maxexp);
    for (ChunkRef ch = src.take(); ch.valid; ch = src.take()) {
        if (ch.by_parts) pack_chunk64_parts(ch, src.merged_codelen(), L, K);
        else if (ch.fast) pack_chunk64<true>(ch, L, K);
        else pack_chunk64<false>(ch, L, K);
    }
    __syncthreads();
    if (lane < K) {
        u64 mn = ~0ull, mx = 0;
#pragma unroll
        for (int k = 0; k < kMmCopies64; ++k) { mn = min(mn, (u64)L.mn[lane * kMmCopies64 + k]); mx = max(mx, (u64)L.mx[lane * kMmCopies64 + k]); }
        if (mn <= mx) { atomicMin(&ext->mmin[lane], mn & 0xFFFFFFFFFFFFFull); atomicMax(&ext->mmax[lane], mx & 0xFFFFFFFFFFFFFull); }
    }
}

// ----------------------------------------------------------------------------- k_spec_sweep
// lc_encode_cached: the single sweep.  Counts the bucket populations like k_hist and, when a cached
// table is in place (ws->spec), codes every chunk with it like k_pack in the same pass over w and
// w_ref.  k_table then either confirms the coding or voids it.
template <int DT>
__global__ __launch_bounds__(64) void k_spec_sweep(const void* __restrict__ w, const void* __restrict__ w_ref, u64 n,
                                                   Workspace* ws, u32* chunk_bits, u32* group_words, u32* prov,
                                                   u32 slot_words, u32 nchunks) {
    __shared__ PackLds L;
    const u32 lane = threadIdx.x;
    const Table& T = ws->table;
    const bool spec = ws->spec != 0;
    for (u32 i = lane; i < 512 * kSpecCopies; i += 64) L.hist[i] = 0;
    if (spec) pack_setup(L, T, lane);
    const u32 K = spec ? T.K : 0;
    __syncthreads();
    VectorChunks src = {w, w_ref, n, prov, slot_words, chunk_bits, group_words, nchunks, K << 3,
                        !spec || T.max_len <= 8, nullptr, 0, 0, nullptr, 16u, 0u, 0u};
    if (!spec) pack_loop<false, DT, 1>(src, L);
    else if (src.row) pack_loop<true, DT, 1>(src, L);
    else pack_loop<true, DT, 0>(src, L);
    __syncthreads();
    for (u32 b = lane; b < 512; b += 64) {
        u32 sum = 0;
#pragma unroll
        for (int k = 0; k < kSpecCopies; ++k) sum += L.hist[hist_slot(b, k)];
        if (sum) atomicAdd(&ws->ext64.hist[(blockIdx.x % kHistCells) * 512 + b], (u64)sum);
    }
    if (spec) pack_merge_extremes(L, ws, K, lane);
}

// ----------------------------------------------------------------------------- k_place
// Builds the chunk area of the blob from the per-chunk slots, one wavefront per chunk.  The
// chunk's word offset is the sum of the record sizes before it (whole groups of 64 chunks from
// group_words, the rest from chunk_bits).  The 64 lane strings are joined without gaps: payload
// word W0 + j of a lane takes the low bits of its word j-1 and the high bits of its word j.
// The payload is assembled in LDS, kPlaceWords words at a time: every lane ORs the words of its shifted string
// that fall into the window into a cleared buffer (so words shared by neighbouring lanes need no special care),
// then the window is written out with coalesced stores.  Most chunks fit one window.  PW words per window: 1024
// lets twice as many workgroups share a compute unit as 2048, which a call with few chunks (all of its workgroups
// resident anyway, one chunk's latency what counts) takes instead.
constexpr u32 kPlaceWords = 1024, kPlaceWordsFew = 2048;

// What the header says of symbol t, held by thread t (of 0 .. 15) of the workgroup that writes it; and of the whole.
struct BlobSymbol { u32 codelen, kept; u64 cnt; u32 mn, mx; u64 mn64, mx64; };      // mn, mx / mn64, mx64: the mantissas' extremes
struct BlobFacts { u32 status, K, k_E, max_len, used_cache, listed; u64 total_words; };

// Representatives (Section 3.1.1: mean of the bucket's largest and smallest member, rounded once
// to fp32, ties to even, done on the mantissas since both share a binade), the header, the last
// offset entry, the result for the host; by a workgroup of at least 128 threads.
__device__ __forceinline__ void write_header(uint8_t* out, const BlobSymbol& my, const BlobFacts& f, Result* host_result,
                                             TableCache* cache, u64 n, int nbits, u32 nchunks, u32 dtype) {
    __shared__ u32 hdr[kHeaderBytes / 4];
    const u32 t = threadIdx.x;
    if (t < kHeaderBytes / 4) hdr[t] = 0;
    __syncthreads();
    const bool ok = f.status == 0;
    const u64 area = chunk_area_of(nchunks);
    const u64 total = ok ? area + 4 * f.total_words : kHeaderBytes;
    if (t == 0) {
        hdr[0] = 0x3142434Cu;                     // "LCB1"
        hdr[1] = 1u | (kHeaderBytes << 16);
        hdr[2] = (u32)n; hdr[3] = (u32)(n >> 32);
        hdr[4] = (u32)nbits;
        hdr[6] = kW; hdr[7] = kV; hdr[8] = kR;
        hdr[10] = (u32)total; hdr[11] = (u32)(total >> 32);
        hdr[12] = f.status;
        hdr[15] = dtype;
        if (ok) { hdr[5] = f.K; hdr[9] = nchunks; hdr[13] = f.k_E; hdr[14] = f.max_len; }
        host_result->bytes = total; host_result->status = f.status; host_result->used_cache = f.used_cache;
        host_result->listed = f.listed; host_result->pad_r = 0;
        if (cache && ok) { cache->valid = 1; cache->nbits = (u32)nbits; cache->K = f.K; cache->pad = 0; }
    }
    if (cache && ok && t < kMaxSym) {              // what this blob was coded with, for the next call
        cache->kept[t] = t < f.K ? my.kept : 0;
        cache->len[t] = t <= f.K ? (my.codelen & 31) : 0;
    }
    if (ok && t <= f.K) {
        const u32 len = my.codelen & 31;
        // representative = midrange of the bucket's extremes, rounded once to nearest even (Section 3.1.1):
        // halve the mantissa sum; an odd sum lies halfway between two mantissas and goes to the even one
        u32 bucket = 0xFFFFu, rep = 0;
        if (t < f.K && dtype != kF64) {
            bucket = my.kept;
            const u32 sum = my.mn + my.mx;
            u32 mm = sum >> 1;
            if ((sum & 1) && (mm & 1)) ++mm;
            rep = (bucket << 23) | mm;
        } else if (t < f.K) {                          // binary64: 52-bit mantissas, high half at header offset 320 + 4 t
            bucket = my.kept;
            const u64 sum = my.mn64 + my.mx64;
            u64 mm = sum >> 1;
            if ((sum & 1) && (mm & 1)) ++mm;
            const u64 rep64 = ((u64)bucket << 52) | mm;
            rep = (u32)rep64;
            hdr[80 + t] = (u32)(rep64 >> 32);
        }
        hdr[16 + 4 * t + 0] = bucket | (len << 16);
        hdr[16 + 4 * t + 1] = rep;
        hdr[16 + 4 * t + 2] = (u32)my.cnt;
        hdr[16 + 4 * t + 3] = (u32)(my.cnt >> 32);
    }
    __syncthreads();
    if (t < kHeaderBytes / 4) reinterpret_cast<u32*>(out)[t] = hdr[t];
    if (ok) {
        // last offset entry and the zero padding of the offset table
        u32* off_tab = reinterpret_cast<u32*>(out + kHeaderBytes);
        const u32 entries = (u32)((area - kHeaderBytes) / 4);
        if (t == 0) off_tab[nchunks] = (u32)f.total_words;
        if (t >= 1 && t < 4 && nchunks + t < entries) off_tab[nchunks + t] = 0;
    }
}

// The header of one vector's blob and the call's outcome for the host, by a workgroup of 256 threads.  group_words: the
// record sizes of the vector's groups of 64 chunks; their sum is the size of the chunk area.  Everything a thread needs
// from memory is asked for before the first use of any of it (the workgroup runs beside a whole placement sweep: every
// dependent round trip costs microseconds there).
__device__ __forceinline__ void finalize_blob(uint8_t* out, EncState* ws, Result* host_result, TableCache* cache,
                                              u64 n, int nbits, u32 nchunks, u32 dtype, const u32* group_words,
                                              const Ext64* ext = nullptr, const u32* bucket_min = nullptr,
                                              const u32* bucket_max = nullptr) {
    __shared__ unsigned long long s_total;
    const u32 t = threadIdx.x;
    const Table& T = ws->table;
    u64 part = 0;
    for (u32 g = t; g < (nchunks + 63) / 64; g += blockDim.x) part += group_words[g];
    if (t == 0) s_total = 0;
    const u32 sym = t < kMaxSym ? t : 0;
    BlobSymbol my = {T.codelen[sym], T.kept[sym], T.cnt[sym], 0x7FFFFFu, 0, 0, 0};
    if (dtype != kF64) {
#pragma unroll
        for (u32 k = 0; k < kExtCopies; ++k) { my.mn = min(my.mn, ws->mmin[k][sym]); my.mx = max(my.mx, ws->mmax[k][sym]); }
        // (an encode with staged keys: the extremes of every bucket were gathered by sweep 1)
        if (bucket_min) { my.mn = bucket_min[my.kept & 511u] & 0x7FFFFFu; my.mx = bucket_max[my.kept & 511u] & 0x7FFFFFu; }
    } else {
        my.mn64 = ext->mmin[sym]; my.mx64 = ext->mmax[sym];
    }
    BlobFacts f = {T.status, T.K, T.k_E, T.max_len, ws->spec_ok, ws->list_count, 0};
    __syncthreads();
    part = wave_sum64(part);
    if (lane_id() == 0 && part) atomicAdd(&s_total, (unsigned long long)part);
    __syncthreads();
    f.total_words = s_total;
    write_header(out, my, f, host_result, cache, n, nbits, nchunks, dtype);
    __syncthreads();
}

// The header of a single vector's blob, the call's outcome for the host, and the scratch state left as the next call
// expects it; by one workgroup of 256 threads.  It runs as the first workgroup of k_place, beside the workgroups that
// place the chunks: everything it needs is final before that kernel starts (table, extremes, and the size of the blob,
// which is the sum of the groups' record sizes), and what it clears none of them reads.  The groups' sums, which they
// do read, are cleared by the next call's first kernel that precedes their use (k_table, or k_spec_table).
__device__ __forceinline__ void finalize_vector(uint8_t* out, Workspace* ws, Result* host_result, const u32* group_words,
                                                TableCache* cache, u64 n, int nbits, u32 nchunks, u32 dtype, int staged) {
    finalize_blob(out, ws, host_result, cache, n, nbits, nchunks, dtype, group_words, &ws->ext64, staged ? ws->bucket_min : nullptr,
                  staged ? ws->bucket_max : nullptr);
    clear_encode_state(ws, nullptr, 0, threadIdx.x, blockDim.x);
    clear_ext64(&ws->ext64, threadIdx.x, blockDim.x);
    if (staged) clear_bucket_extremes(ws, threadIdx.x, blockDim.x);
    // (no fence: the host reads its result after waiting for the stream, and the end of the kernel makes every store
    // visible; a system-scope fence here would have to write back what the other workgroups have just placed)
}

// Chunk c of one vector, by one wavefront of a workgroup of four; `valid` false: an idle wavefront.
template <u32 PW>
__device__ __forceinline__ void place_chunk(uint8_t* out, EncState* ws, const u32* __restrict__ chunk_bits,
                                            const u32* __restrict__ group_words, const u32* __restrict__ prov,
                                            u32 slot_words, u32 nchunks, u32 c, bool valid) {
    __shared__ u32 s_buf_all[4][PW];
    const u32 lane = lane_id(), wv = threadIdx.x >> 6;
    u32* s_buf = s_buf_all[wv];
    const u32* slot = prov + (u64)(valid ? c : 0) * slot_words;
    const u32 own = valid ? __builtin_amdgcn_readfirstlane(chunk_bits[c]) : 0;
    const bool merged = (own & kMergedChunk) != 0;               // wave-uniform: no slot, 256 copies of one code per lane
    const bool record = valid && (own & (kMergedChunk | kRawChunk)) == 0;      // the slot holds the record as it is
    const u32 bits = !valid || record ? 0 : merged ? (own & kChunkBits) / kW : reinterpret_cast<const uint16_t*>(slot)[lane];
    const u32 g = c >> 6;
    u64 part = (valid && 64 * g + lane < c) ? kLaneBitsWords + (((chunk_bits[64 * g + lane] & kChunkBits) + 31) >> 5) : 0;
    if (valid) {
#pragma unroll 4
        for (u32 j = lane; j < g; j += kW) part += group_words[j];
    }
    const u64 word_off = wave_sum64(part);
    if (record) {
        // 16-byte vectors from the slot to a place in the blob that is aligned to words only, eight in flight per lane
        typedef u32x4 __attribute__((aligned(4))) u32x4_word;
        const u32 nw = kLaneBitsWords + (((own & kChunkBits) + 31) >> 5), nvec = nw >> 2;
        u32* to = reinterpret_cast<u32*>(out + chunk_area_of(nchunks)) + word_off;
        const u32x4* from = reinterpret_cast<const u32x4*>(slot);
        for (u32 i0 = 0; i0 < nvec; i0 += 8 * kW) {
            u32x4 x[8];
#pragma unroll
            for (u32 k = 0; k < 8; ++k) if (i0 + k * kW + lane < nvec) x[k] = from[i0 + k * kW + lane];
#pragma unroll
            for (u32 k = 0; k < 8; ++k) if (i0 + k * kW + lane < nvec) reinterpret_cast<u32x4_word*>(to)[i0 + k * kW + lane] = x[k];
        }
        if (lane < (nw & 3)) to[4 * nvec + lane] = slot[4 * nvec + lane];
        if (lane == 0) reinterpret_cast<u32*>(out + kHeaderBytes)[c] = (u32)word_off;
        return;
    }
    const u32 incl = wave_incl_scan(bits);
    const u32 o = incl - bits;                               // first bit of this lane's string
    const u32 total_bits = __shfl(incl, 63, 64);
    const u32 nwords = (total_bits + 31) >> 5;
    uint8_t* rec = out + chunk_area_of(nchunks) + 4 * word_off;
    u32* payload = reinterpret_cast<u32*>(rec + 2 * kW);
    if (valid) {
        reinterpret_cast<uint16_t*>(rec)[lane] = (uint16_t)bits;
        if (lane == 0) {
            reinterpret_cast<u32*>(out + kHeaderBytes)[c] = (u32)word_off;
        }
    }
    if (merged) {
        // every lane's string is a whole number of codes and of words, so the payload is the code repeated
        // 16384 times: word i holds the 32 bits from bit 32 i of that endless repetition on
        const u32 codelen = __builtin_amdgcn_readfirstlane(ws->table.codelen[ws->table.K]);
        const u32 len = max(codelen & 31, 1u);                  // (a merged symbol that occurs has a code)
        u64 rep = (u64)(codelen >> 5) << (64 - len);            // the code repeated from bit 63 downwards
        for (u32 filled = len; filled < 64; filled <<= 1) rep |= rep >> filled;
        u32 phase = (32 * lane) % len;                          // bit of the code that word i starts with
        const u32 step = (32 * kW) % len;
        for (u32 i = lane; i < nwords; i += kW) {
            payload[i] = (u32)((rep << phase) >> 32);
            phase += step;
            if (phase >= len) phase -= len;
        }
    }
    const u32 sh = o & 31, W0 = o >> 5, nloc = (bits + 31) >> 5;
    const u32 nt = (bits && !merged) ? ((o + bits - 1) >> 5) - W0 + 1 : 0;   // payload words this lane touches
    const u32* lane_words = slot + kLaneBitsWords + lane;
    if (merged) return;
    // Only this wavefront touches its buffer, and a wavefront's LDS operations take effect in program order: no
    // barrier between clearing, ORing and reading a window.
    for (u32 win = 0; win < nwords; win += PW) {
        const u32 wlen = min(PW, nwords - win);
        for (u32 i = lane; i < wlen; i += kW) s_buf[i] = 0;
        // the touched words j of this lane (payload word W0 + j) that lie inside the window
        const u32 jlo = win > W0 ? win - W0 : 0;
        const u32 jend = win + wlen > W0 ? win + wlen - W0 : 0;
        const u32 jhi = jend < nt ? jend : nt;
        const u32 cnt = jhi > jlo ? jhi - jlo : 0;
        const u32 cnt_max = wave_max_u32(cnt);
        u32 prev = (cnt != 0 && jlo != 0) ? lane_words[(jlo - 1) * kW] : 0;   // (jlo - 1 < nloc whenever jlo < nt)
        for (u32 i0 = 0; i0 < cnt_max; i0 += 8) {
            u32 buf[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const u32 j = jlo + i0 + k;
                buf[k] = (i0 + k < cnt && j < nloc) ? lane_words[j * kW] : 0;
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                if (i0 + k < cnt) {
                    const u32 val = __builtin_amdgcn_alignbit(prev, buf[k], sh);
                    prev = buf[k];
                    atomicOr(&s_buf[W0 + jlo + i0 + k - win], val);
                }
            }
        }
        for (u32 i = lane; i < wlen; i += kW) payload[win + i] = s_buf[i];
    }
}

// Workgroup 0 writes the header and reports the outcome (finalize_vector); the others place four chunks each.
struct FinalizeArgs { Result* host_result; TableCache* cache; u64 n; int nbits; u32 dtype; int staged; };

template <u32 PW>
__global__ __launch_bounds__(256) void k_place(uint8_t* out, Workspace* ws, const u32* __restrict__ chunk_bits,
                                               const u32* __restrict__ group_words, const u32* __restrict__ prov,
                                               u32 slot_words, u32 nchunks, u32* chunk_maxexp, FinalizeArgs fin) {
    if (blockIdx.x == 0) {
        finalize_vector(out, ws, fin.host_result, group_words, fin.cache, fin.n, fin.nbits, nchunks, fin.dtype, fin.staged);
        return;
    }
    const u32 c = (blockIdx.x - 1) * 4 + (threadIdx.x >> 6);
    // sweep 2 was the last to look at the chunk maxima: leave them cleared for the next call, whatever this one's outcome
    if (c < nchunks && lane_id() == 0) chunk_maxexp[maxexp_slot(c)] = 0;
    // the last workgroup may hold idle wavefronts
    place_chunk<PW>(out, ws, chunk_bits, group_words, prov, slot_words, nchunks, c, c < nchunks && ws->table.status == 0);
}

// ----------------------------------------------------------------------------- k_encode_one
// A short vector in one launch: a workgroup per chunk, all of them resident together, that keeps its deltas in registers
// from the count to the code.  What such a call costs in four kernels is not bytes but their starts, the gaps between them
// and every chunk's round trips to memory (chunk maxima, table, slot, slot again): 2^20 fp32 elements 7.0 + 4.6 + 7.9 + 3.7
// us and three gaps, 40.8 us the call (15.2 and 28.5 so).  Here the workgroups meet twice: when all counts are in (each then builds the table for itself, from
// the same counts), and when all record sizes are known (each then knows where its record goes); see GridMeeting.
// A cached table's lengths (lc_encode_cached; see k_spec_table), by one wavefront, lane j holding symbol j: whether the cache
// is usable.
__device__ __forceinline__ bool cached_table(const TableCache* cache, int nbits, u32* kept, u32* len) {
    const u32 lane = lane_id(), K = cache->K;
    const u32 kmax = (1u << nbits) - 1;
    if (cache->valid != 1 || cache->nbits != (u32)nbits || K > kmax) return false;
    const u32 b = lane < K ? cache->kept[lane] : 0u, e = b & 255u, l = lane <= K ? cache->len[lane] : 0u;
    const u32 order = (e << 1) | (1u - ((b >> 8) & 1u));             // larger exponent first, + before -
    const u32 before = __shfl_up(order, 1, 64);
    bool bad = lane < K && (b >= 512u || e == 0 || e == 255u || (lane > 0 && order >= before));
    bad = bad || l > 15;
    const u32 active = (u32)__popcll(__ballot(l != 0)), kraft = wave_sum32(l && l <= 15 ? 1u << (15 - l) : 0u);
    if (__any(bad) || (active >= 2 && kraft != (1u << 15)) || (active == 1 && kraft != (1u << 14))) return false;
    *kept = b; *len = l;
    return true;
}

struct OneArgs {
    const void* w; const void* w_ref; u64 n;
    uint8_t* out; Workspace* ws; u32* record_words; TableCache* cache; Result* host_result;
    u64 goal[kMeetLines];
    u32 nchunks, lines, limit;
    int nbits;
};
constexpr u32 kOneCopies = 16;      // LDS copies of the chunk's counts (8 of them serve a wavefront in twice the time: it is not
                                    // hidden behind a stream here), then 8 of the buckets' smallest and largest patterns
constexpr u32 kAbsent = 0xFFFFFFFFu;    // the delta that stands for what a ragged chunk lacks: of a bucket that no vector that is coded holds

template <int DT>
__global__ __launch_bounds__(kWgThreads, 4) void k_encode_one(OneArgs a) {
    typedef typename Raw<DT>::type raw_t;
    __shared__ PackWg L;
    __shared__ TableLds<8> S;
    __shared__ u32 s_go, s_max_len, s_reuse, s_cached, s_cached_kept[kMaxSym], s_cached_len[kMaxSym], s_codelen[kMaxSym];
    __shared__ u32 s_before[kWgWaves], s_all[kWgWaves];
    // the counts and extremes lie where the coding's tables and areas go later
    static_assert(sizeof(PackWg) >= 4 * 512 * kOneCopies && alignof(PackWg) >= 16, "room for the counts");
    static_assert(2 * (sizeof(PackWg) + sizeof(TableLds<8>) + 2560) <= kLdsPerCu, "two workgroups per compute unit: the host counts on that many being resident");
    u32* const area = reinterpret_cast<u32*>(&L);
    Workspace* ws = a.ws;
    const u64 n = a.n;
    const u32 t = threadIdx.x, lane = lane_id(), v = __builtin_amdgcn_readfirstlane(t >> 6), c = blockIdx.x, first_row = kWgRows * v;
    const bool full = (u64)(c + 1) * kChunk <= n;
    GridMeeting meet = {ws->meeting(), 0, a.lines, a.limit};
#pragma unroll
    for (u32 k = 0; k < kMeetLines; ++k) meet.goal = lane == k ? a.goal[k] : meet.goal;
    auto fill = [&](u32 from, u32 count, u32 value) {
        const u32x4 x = {value, value, value, value};
        for (u32 i = t; i < count / 4; i += kWgThreads) reinterpret_cast<u32x4*>(area + from)[i] = x;
    };
    // ---- this wavefront's 8 rows, as deltas
    u32 u[kWgRows * kV];
    {
        raw_t A[kWgRows], B[kWgRows];
        if (full) {
#pragma unroll
            for (u32 k = 0; k < kWgRows; ++k) { A[k] = load_raw_any<DT>(a.w, row_at(c, first_row + k)); B[k] = load_raw_any<DT>(a.w_ref, row_at(c, first_row + k)); }
        } else {
#pragma unroll
            for (u32 k = 0; k < kWgRows; ++k) {
                const u64 i = row_at(c, first_row + k);
                const bool whole = i - lane * kV + kRowElems <= n;          // (the same in every lane)
                A[k] = whole ? load_raw_any<DT>(a.w, i) : load_raw_guarded<DT>(a.w, i, n);
                B[k] = whole ? load_raw_any<DT>(a.w_ref, i) : load_raw_guarded<DT>(a.w_ref, i, n);
            }
        }
        fill(0, 512 * kOneCopies, 0);
        if (v == 1 && a.cache) {
            u32 kept = 0, len = 0;
            const bool ok = cached_table(a.cache, a.nbits, &kept, &len);
            if (lane < kMaxSym) { s_cached_kept[lane] = kept; s_cached_len[lane] = len; }
            if (lane == 0) s_cached = ok ? a.cache->K + 1 : 0;
        }
#pragma unroll
        for (u32 k = 0; k < kWgRows; ++k) {
            float xa[4], xb[4];
            unpack<DT>(A[k], xa); unpack<DT>(B[k], xb);
#pragma unroll
            for (u32 e = 0; e < kV; ++e) u[kV * k + e] = delta_bits(xa[e], xb[e]);
        }
        if (!full) {
#pragma unroll
            for (u32 i = 0; i < kWgRows * kV; ++i) if (row_at(c, first_row + i / kV) + i % kV >= n) u[i] = kAbsent;
        }
    }
    __syncthreads();
#pragma unroll
    for (u32 i = 0; i < kWgRows * kV; ++i) atomicAdd(&area[(u[i] >> 23) * kOneCopies + (lane & (kOneCopies - 1))], 1u);
    __syncthreads();
    {
        u32 sum = 0;
#pragma unroll
        for (u32 k = 0; k < kOneCopies / 4; ++k) { const u32x4 x = reinterpret_cast<const u32x4*>(area)[t * (kOneCopies / 4) + k]; sum += x.x + x.y + x.z + x.w; }
        if (t == kAbsent >> 23 && (u64)(c + 1) * kChunk > n) sum -= (u32)((u64)(c + 1) * kChunk - n);
        if (sum) atomicAdd(&ws->ext64.hist[(c % kHistCells) * 512 + t], (u64)sum);
    }
    wait_own_operations();
    __syncthreads();
    if (t == 0) meet.arrive(0);
    // meanwhile the extremes of this chunk's buckets (Section 3.1.1: a representative is the mean of the two), 8 copies
    constexpr u32 kExt = 8;
    fill(0, 512 * kExt, 0xFFFFFFFFu); fill(512 * kExt, 512 * kExt, 0);
    __syncthreads();
    // (zeros and subnormals are never kept, and of a vector that has not changed every lane would queue for the same word: 2^20
    // fp32 elements 28.9 -> 26.6 us, 2^23 45.3 -> 42.6.  The extremes by symbol while coding instead, 32 copies of them: 2^22
    // fp32 elements 30.6 -> 34.5 us, 2^23 45.4 -> 49.9.)
#pragma unroll
    for (u32 i = 0; i < kWgRows * kV; ++i) {
        const u32 at = (u[i] >> 23) * kExt + (lane & (kExt - 1));
        if ((u[i] & 0x7F800000u) != 0) { atomicMin(&area[at], u[i]); atomicMax(&area[512 * kExt + at], u[i]); }
    }
    // ---- all counts are in
    if (v == 0) { const bool go = meet.wait(0); if (lane == 0) s_go = go ? 1u : 0u; }
    __syncthreads();
    if (!s_go) return;
    const u32 kmax = (1u << a.nbits) - 1;
    u64 part[kHistCells], cnt[1] = {0};
#pragma unroll
    for (u32 k = 0; k < kHistCells; ++k) part[k] = load_shared(&ws->ext64.hist[k * 512 + bucket_at<8>(t)]);
#pragma unroll
    for (u32 k = 0; k < kHistCells; ++k) cnt[0] += part[k];
    const u32 candidates = rank_buckets<8>(S, cnt, kmax), K = candidates < kmax ? candidates : kmax;
    __syncthreads();
    if (v == 0) {
        // the code, as in table_build
        const u64 own = symbol_count(S.cnt, K, n);
        const u32 nl = (u32)__popcll(__ballot(own != 0));
        u32 len = 0;
        bool reuse = false;
        if (a.cache && s_cached != 0) {
            const u32 cached_len = lane <= K ? s_cached_len[lane] : 0u;
            const bool differs = (lane < K && s_cached_kept[lane] != S.kept[lane]) || (lane <= K && (cached_len != 0) != (own != 0));
            const u64 payload_bits = wave_sum64(own * cached_len);
            reuse = S.nonfinite == 0 && s_cached == K + 1 && !__any(differs) && payload_bits <= n * (u64)a.nbits;
            if (reuse) len = cached_len;
        }
        if (!reuse && nl == 1) len = own != 0 ? 1u : 0u;
        if (!reuse && nl >= 2) len = code_lengths((u32)own);
        const u32 code = canonical_code(len), max_len = wave_max_u32(len);
        if (lane < kMaxSym) s_codelen[lane] = lane <= K ? ((code << 5) | len) : 0u;
        if (lane == K) S.cnt[lane] = own;
        if (lane == 0) { s_max_len = max_len; s_reuse = reuse ? 1u : 0u; }
    } else if (v <= kMaxSym * kExt / kW) {
        // the extremes of the kept buckets, 8 lanes to a symbol, to one of kExtCopies copies (see pack_merge_extremes)
        const u32 i = t - kW, sym = i / kExt, at = (sym < K ? S.kept[sym] : 0u) * kExt + i % kExt;
        u32 mn = area[at], mx = area[512 * kExt + at];
#pragma unroll
        for (int d = 1; d < (int)kExt; d <<= 1) { mn = min(mn, (u32)__shfl_xor(mn, d, 64)); mx = max(mx, (u32)__shfl_xor(mx, d, 64)); }
        const u32 copy = c % kExtCopies;
        if (i % kExt == 0 && sym < K && mn <= mx) { atomicMin(&ws->mmin[copy][sym], mn & 0x7FFFFFu); atomicMax(&ws->mmax[copy][sym], mx & 0x7FFFFFu); }
    }
    __syncthreads();
    const bool finite = S.nonfinite == 0;
    const u32 sy = S.sym[t] == 0xFF ? K : S.sym[t];
    L.sym8[t] = (uint8_t)((t == kAbsent >> 23 ? kMaxSym : sy) << 3);
    pair_setup(L, s_codelen);
    if (t < kMaxSym) L.codelen[t] = s_codelen[t];
    if (t == 0) L.overflow = 0;
    for (u32 i = t; i < kPayloadWords; i += kWgThreads) L.payload[i] = 0;
    __syncthreads();
    // ---- this chunk's code (of a vector with a delta that is not finite there is none)
    LanePart P;
    P.start(L, v);
    if (finite) {
#pragma unroll
        for (u32 i = 0; i < kWgRows * kV; i += 8) {
            u32 sym[8];
#pragma unroll
            for (u32 k = 0; k < 8; ++k) sym[k] = L.sym8[u[i + k] >> 23];
            code_symbols(sym, L, P);
        }
    }
    const PartPlaces at = part_places(P, v, L);
    if (t == 0) __hip_atomic_store(&a.record_words[c], kLaneBitsWords + at.nwords, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    wait_own_operations();
    __syncthreads();
    // ---- all sizes and extremes are known
    if (t == 0) meet.arrive(1);
    if (!at.overflow) join_parts(at, v, L);
    if (v == 0) { const bool go = meet.wait(1); if (lane == 0) s_go = go ? 1u : 0u; }
    __syncthreads();
    if (!s_go) return;
    const u32 sym = t < kMaxSym ? t : 0;
    BlobSymbol my = {s_codelen[sym], S.kept[sym], S.cnt[sym], 0x7FFFFFu, 0, 0, 0};
    if (c == 0 && t < kMaxSym) {
#pragma unroll
        for (u32 k = 0; k < kExtCopies; ++k) { my.mn = min(my.mn, load_shared(&ws->mmin[k][sym])); my.mx = max(my.mx, load_shared(&ws->mmax[k][sym])); }
    }
    u32 before = 0, all = 0;
    for (u32 i = t; i < a.nchunks; i += kWgThreads) { const u32 words = load_shared(&a.record_words[i]); all += words; before += i < c ? words : 0u; }
    before = wave_sum32(before); all = wave_sum32(all);
    if (lane == 0) { s_before[v] = before; s_all[v] = all; }
    __syncthreads();
    before = 0; all = 0;
#pragma unroll
    for (u32 k = 0; k < kWgWaves; ++k) { before += s_before[k]; all += s_all[k]; }
    if (c == 0) {
        // the first workgroup: the header, the outcome, and the scratch state as the next call expects it (the others are
        // through with the counts, and only it reads the extremes)
        const BlobFacts f = {finite ? 0u : 2u, K, candidates + S.zero_class, s_max_len, s_reuse, a.nchunks, all};
        write_header(a.out, my, f, a.host_result, a.cache, n, a.nbits, a.nchunks, (u32)DT);
        for (u32 i = t; i < kBuckets64 / 2; i += kWgThreads) reinterpret_cast<ulonglong2*>(ws->ext64.hist)[i] = make_ulonglong2(0, 0);
        clear_extremes(ws, t, kWgThreads);
    }
    if (!finite) return;
    u32* rec = reinterpret_cast<u32*>(a.out + chunk_area_of(a.nchunks)) + before;
    if (v == 0) reinterpret_cast<uint16_t*>(rec)[lane] = (uint16_t)at.bits;
    if (t == 0) reinterpret_cast<u32*>(a.out + kHeaderBytes)[c] = before;
    if (!at.overflow) { copy_payload(rec + kLaneBitsWords, at.nwords, L); return; }
    PartSymbols Q;
    Q.count = 0;
#pragma unroll
    for (u32 i = 0; i < kWgRows * kV; ++i) {
        if (i % 16 == 0) Q.s[i / 16] = 0;
        Q.s[i / 16] |= (u64)((L.sym8[u[i] >> 23] >> 3) & 15u) << (4 * (i % 16));
        Q.count += u[i] != kAbsent ? 1u : 0u;                     // (those past the vector's end are a lane's last)
    }
    finish_long(rec + kLaneBitsWords, Q, at.o, at.nwords, L);
}

// ----------------------------------------------------------------------------- batched encode
// lc_encode_batch: many vectors, one table each, in five launches, six where the chunks to read are listed.  The chunks of all
// tensors are numbered through; the counting and the coding sweep are a workgroup per chunk.
// One workgroup per tensor: what the host says about it (read from mapped host memory, kept for the kernels behind this one: a
// copy of the list to the device ahead of the call took longer than that read: 161 tensors 129 -> 125 us), which chunks are
// its own, its groups and its state cleared.
__global__ __launch_bounds__(256) void kb_setup(BatchArgs a) {
    __shared__ Seg sg;
    const u32 t = threadIdx.x, sidx = blockIdx.x;
    EncState& st = a.states[sidx];
    // (one read of it per workgroup)
    if (t < sizeof(Seg) / 4) reinterpret_cast<u32*>(&sg)[t] = reinterpret_cast<const u32*>(a.host_segs + sidx)[t];
    constexpr u32 kExt = kExtCopies * kMaxSym;
    for (u32 i = t; i < 512; i += 256) st.hist[i] = 0;
    for (u32 i = t; i < kExt; i += 256) { (&st.mmin[0][0])[i] = 0x7FFFFFu; (&st.mmax[0][0])[i] = 0; }
    if (t == 0) { st.spec = 0; st.spec_ok = 0; st.table.status = 0; }
    if (t == 0 && sidx == 0) *a.list_count = 0;
    __syncthreads();
    if (t < sizeof(Seg) / 4) reinterpret_cast<u32*>(a.segs + sidx)[t] = reinterpret_cast<const u32*>(&sg)[t];
    for (u32 c = t; c < sg.nchunks; c += 256) a.seg_of_chunk[sg.chunk0 + c] = sidx;
    for (u32 g = t; g < (sg.nchunks + 63) / 64; g += 256) a.group_words[sg.group0 + g] = 0;
}

// The counting sweep of a batched call: a workgroup of 8 wavefronts per chunk, whose loads are all on their way at once, or
// (STAY) per `run` chunks in a row, whose counts it hands in together where they are one tensor's.  Arrays off alignment take the
// same loads.  Against a wavefront per chunk, whole calls (with the two codes per append of then), us: 161 tensors of 25.6 M fp32
// 117 -> 113, 32 of 138 M 268 -> 249, 60 of 2^25 bf16 130 -> 105, off alignment fp32 200 -> 160, bf16 353 -> 152.
// It also notes the largest |delta| exponent of every chunk and of each of its 4 KiB parts: from these the chunks that hold
// merged elements only are told before the coding sweep, and of a mostly merged chunk the parts that have to be read.
// SHORT: for tensors of a few rows.  Wavefronts without a row leave theirs alone, and rows are read by parts, so that a fourth
// workgroup of fp32 fits a compute unit beside three: 1,000 tensors of 64 elements 89.0 us the call by the other form, whose last
// workgroups wait for a second round, 83.3 so (a wavefront per chunk 84.5); bf16 84.7 and 82.8; of 8,000 elements 110 and 105.5,
// 105.8 and 104.0.
template <int DT, bool STAY, bool SHORT = false>
__global__ __launch_bounds__(kWgThreads, SHORT ? 8 : 4) void kb_hist(BatchArgs a, u32 run) {
    typedef typename Raw<DT>::type raw_t;
    constexpr u32 kCopies = 16, kPartRows = 4096 / (kRowElems * elem_bytes<DT>());      // 4 rows per 4 KiB part, or 8
    __shared__ alignas(16) u32 hist[512 * kCopies];
    __shared__ u32 s_largest[kWgWaves];
    const u32 t = threadIdx.x, lane = lane_id(), v = __builtin_amdgcn_readfirstlane(t >> 6), first_row = kWgRows * v;
    const u32 first = blockIdx.x * (STAY ? run : 1u), end = STAY ? min(first + run, a.total_chunks) : first + 1;
    for (u32 i = t; i < 512 * kCopies / 4; i += kWgThreads) reinterpret_cast<u32x4*>(hist)[i] = u32x4{0, 0, 0, 0};
    u32 sidx = load_uniform(a.seg_of_chunk + first);
#pragma unroll 1
    for (u32 g = first; g < end; ++g) {
        const u32 next = g + 1 < end ? load_uniform(a.seg_of_chunk + g + 1) : 0xFFFFFFFFu;
        const Seg& sg = a.segs[sidx];
        const u64 n = sg.n;
        const u32 c = g - sg.chunk0;
        const bool full = (u64)(c + 1) * kChunk <= n;
        u32 largest = 0;
        if constexpr (SHORT) {
            __syncthreads();
#pragma unroll 1
            for (u32 part = 0; part < kWgRows / kPartRows; ++part) {
                const u32 r0 = first_row + part * kPartRows;
                u32 most = 0;
                if ((u64)c * kChunk + r0 * kRowElems < n) {
                    raw_t A[kPartRows], B[kPartRows];
#pragma unroll
                    for (u32 k = 0; k < kPartRows; ++k) {
                        const u64 i = row_at(c, r0 + k);
                        const bool whole = i - lane * kV + kRowElems <= n;      // (the same in every lane)
                        A[k] = whole ? load_raw_any<DT>(sg.w, i) : load_raw_guarded<DT>(sg.w, i, n);
                        B[k] = whole ? load_raw_any<DT>(sg.w_ref, i) : load_raw_guarded<DT>(sg.w_ref, i, n);
                    }
#pragma unroll
                    for (u32 k = 0; k < kPartRows; ++k) {
                        float xa[4], xb[4];
                        unpack<DT>(A[k], xa); unpack<DT>(B[k], xb);
#pragma unroll
                        for (u32 e = 0; e < kV; ++e) {
                            const u32 u = delta_bits(xa[e], xb[e]);
                            if (row_at(c, r0 + k) + e < n) {
                                atomicAdd(&hist[(u >> 23) * kCopies + (lane & (kCopies - 1))], 1u);
                                most = max(most, u & 0x7FFFFFFFu);
                            }
                        }
                    }
                    most = wave_max_u32(most) >> 23;
                }
                if (lane == 0) a.part_max[(u64)g * kPartBytes + first_row / kPartRows + part] = (uint8_t)most;
                largest = max(largest, most);
            }
        } else {
            raw_t A[kWgRows], B[kWgRows];
            if (full) {
#pragma unroll
                for (u32 k = 0; k < kWgRows; ++k) { A[k] = load_raw_any<DT>(sg.w, row_at(c, first_row + k)); B[k] = load_raw_any<DT>(sg.w_ref, row_at(c, first_row + k)); }
            } else {
#pragma unroll
                for (u32 k = 0; k < kWgRows; ++k) {
                    const u64 i = row_at(c, first_row + k);
                    const bool whole = i - lane * kV + kRowElems <= n;              // (the same in every lane)
                    A[k] = whole ? load_raw_any<DT>(sg.w, i) : load_raw_guarded<DT>(sg.w, i, n);
                    B[k] = whole ? load_raw_any<DT>(sg.w_ref, i) : load_raw_guarded<DT>(sg.w_ref, i, n);
                }
            }
            __syncthreads();                             // (the counts are cleared, the last chunk's maxima read)
#pragma unroll
            for (u32 part = 0; part < kWgRows / kPartRows; ++part) {
                u32 most = 0;
#pragma unroll
                for (u32 k = part * kPartRows; k < (part + 1) * kPartRows; ++k) {
                    float xa[4], xb[4];
                    unpack<DT>(A[k], xa); unpack<DT>(B[k], xb);
#pragma unroll
                    for (u32 e = 0; e < kV; ++e) {
                        const u32 u = delta_bits(xa[e], xb[e]);
                        if (full || row_at(c, first_row + k) + e < n) {
                            atomicAdd(&hist[(u >> 23) * kCopies + (lane & (kCopies - 1))], 1u);
                            most = max(most, u & 0x7FFFFFFFu);
                        }
                    }
                }
                most = wave_max_u32(most) >> 23;
                if (lane == 0) a.part_max[(u64)g * kPartBytes + first_row / kPartRows + part] = (uint8_t)most;
                largest = max(largest, most);
            }
        }
        if (lane == 0) s_largest[v] = largest;
        __syncthreads();
        if (t == 0) {
#pragma unroll
            for (u32 k = 0; k < kWgWaves; ++k) largest = max(largest, s_largest[k]);
            a.chunk_maxexp[g] = largest;
        }
        if (next != sidx) {
            u32 sum = 0;
#pragma unroll
            for (u32 k = 0; k < kCopies / 4; ++k) {
                u32x4* x = reinterpret_cast<u32x4*>(hist) + t * (kCopies / 4) + k;
                sum += x->x + x->y + x->z + x->w;
                if (STAY) *x = u32x4{0, 0, 0, 0};
            }
            if (sum) atomicAdd(&a.states[sidx].hist[t], (u64)sum);
        }
        sidx = next;
    }
}

__global__ __launch_bounds__(table_threads<8>()) void kb_table(BatchArgs a) {
    table_build<8>(&a.states[blockIdx.x], nullptr, a.segs[blockIdx.x].n, a.nbits, nullptr, 0, nullptr, nullptr);
}

// Between the tables and the coding sweep: which chunks that sweep has to read.  A full chunk whose largest exponent
// lies below every kept bucket of its tensor holds the merged symbol 16384 times (Section 3.1.1): it gets its size and
// the flag that lets kb_place write the repeated code, and stays off the list; all others are listed, in no particular
// order (one claim on the list per wavefront).
__global__ __launch_bounds__(256) void kb_list(BatchArgs a) {
    const u32 g = blockIdx.x * blockDim.x + threadIdx.x, lane = lane_id();
    bool listed = false;
    u32 group = 0xFFFFFFFFu, words = 0;
    if (g < a.total_chunks) {
        const u32 sidx = a.seg_of_chunk[g];
        const Seg& sg = a.segs[sidx];
        const Table& T = a.states[sidx].table;
        const u32 c = g - sg.chunk0;
        const bool merged = T.status == 0 && (u64)(c + 1) * kChunk <= sg.n && a.chunk_maxexp[g] < T.min_kept_exp;
        listed = !merged;
        if (merged) {
            const u32 len_merged = T.codelen[T.K] & 31;
            a.chunk_bits[g] = kMergedChunk | (kChunk * len_merged);
            group = sg.group0 + (c >> 6);
            words = kLaneBitsWords + kChunk / 32 * len_merged;
        }
    }
    // the merged chunks' records go into their groups' sums, one addition per group that the wavefront's chunks touch
    // (a group belongs to one tensor, so its merged chunks have records of one size)
    for (u64 pending = __ballot(group != 0xFFFFFFFFu); pending != 0;) {
        const u32 first = (u32)__ffsll((unsigned long long)pending) - 1;
        const u32 key = read_lane(group, first);
        const u64 same = __ballot(group == key);
        if (lane == first) atomicAdd(&a.group_words[key], (u32)__popcll(same) * words);
        pending &= ~same;
    }
    const u64 m = __ballot(listed);
    if (m == 0) return;
    u32 base = 0;
    if (lane == 0) base = atomicAdd(a.list_count, (u32)__popcll(m));
    base = __builtin_amdgcn_readfirstlane(base);
    if (listed) a.chunk_list[base + (u32)__popcll(m & ((1ull << lane) - 1))] = g;
}

// The coding sweep: a workgroup per chunk of the list, as k_pack.
template <int DT>
__global__ __launch_bounds__(kWgThreads, DT == kF32 ? 4 : 8) void kb_pack(BatchArgs a) {
    __shared__ PackWg L;
    u32 g = blockIdx.x;
    if (a.listed) {
        if (g >= load_uniform(a.list_count)) return;
        g = load_uniform(a.chunk_list + g);
    }
    const u32 sidx = __builtin_amdgcn_readfirstlane(a.seg_of_chunk[g]);
    const Seg& sg = a.segs[sidx];
    EncState* st = &a.states[sidx];
    ChunkRef ch;
    ch.c = g - sg.chunk0;
    ch.w = sg.w; ch.w_ref = sg.w_ref; ch.n = sg.n;
    ch.slot = a.prov + (u64)g * a.slot_words; ch.bits_at = a.chunk_bits + g; ch.group_at = a.group_words + sg.group0 + (ch.c >> 6);
    ch.fast = (u64)(ch.c + 1) * kChunk <= sg.n;
    if (st->table.status != 0) return;                 // (a delta that is not finite: a header-only blob)
    const u32 largest = load_uniform(a.chunk_maxexp + g), maxima = part_word<DT>(a.part_max + (u64)g * kPartBytes);
    if (!a.listed && noted_as_merged(ch, st->table, largest)) return;
    pack_chunk_wg<DT>(ch, st->table, maxima, st, L);
}

// The first `count` workgroups write the tensors' headers and report their outcomes (everything that takes is final
// before the placement starts, as for a single vector: see finalize_vector); the others place four chunks each.
__global__ __launch_bounds__(256) void kb_place(BatchArgs a) {
    if (blockIdx.x < a.count) {
        const Seg& sg = a.segs[blockIdx.x];
        finalize_blob(sg.out, &a.states[blockIdx.x], &a.results[blockIdx.x], nullptr, sg.n, a.nbits, sg.nchunks, (u32)a.dtype,
                      a.group_words + sg.group0);
        return;
    }
    const u32 g = (blockIdx.x - a.count) * 4 + (threadIdx.x >> 6);
    const bool in_range = g < a.total_chunks;
    const u32 sidx = in_range ? a.seg_of_chunk[g] : 0;
    const Seg& sg = a.segs[sidx];
    EncState* st = &a.states[sidx];
    place_chunk<kPlaceWords>(sg.out, st, a.chunk_bits + sg.chunk0, a.group_words + sg.group0, a.prov + (u64)sg.chunk0 * a.slot_words,
                a.slot_words, sg.nchunks, in_range ? g - sg.chunk0 : 0, in_range && st->table.status == 0);
}

// ----------------------------------------------------------------------------- launchers
void launch_reset(Workspace* ws, uint32_t* group_words, uint32_t* chunk_maxexp, hipStream_t s) {
    hipLaunchKernelGGL(k_reset, dim3(1), dim3(1024), 0, s, ws, group_words, (u32)kMaxGroups, chunk_maxexp, (u32)kMaxChunks);
}

void launch_reset_one(Workspace* ws, hipStream_t s) { hipLaunchKernelGGL(k_reset_one, dim3(1), dim3(1024), 0, s, ws); }

void launch_reset_chunks(Workspace* ws, uint32_t* group_words, uint32_t* chunk_maxexp, uint32_t nchunks, hipStream_t s) {
    hipLaunchKernelGGL(k_reset_chunks, dim3(1), dim3(1024), 0, s, ws, group_words, (nchunks + 63) / 64, chunk_maxexp, nchunks);
}

// keys.exp != null: stage keys (binary32)
void launch_hist(const void* w, const void* w_ref, uint64_t n, int dtype, Workspace* ws, uint32_t* chunk_maxexp, uint8_t* batch_max,
                 KeyPlanes keys, const Tuning& tune, hipStream_t s) {
    if (n == 0) return;
    const u32 threads = tune.hist_threads;
    const u64 units = n / (dtype == kF32 ? 4 : dtype == kF64 ? 2 : 8);   // 16-byte units
    u64 blocks = (units + 4 * threads - 1) / (4 * threads);
    const u64 cap = (u64)tune.num_cu * tune.hist_blocks_per_cu;
    if (blocks > cap) blocks = cap;
    if (blocks < 1) blocks = 1;
    if (dtype == kF64) {
        uint16_t* part_max = reinterpret_cast<uint16_t*>(batch_max);
        hipLaunchKernelGGL(k_hist64, dim3((u32)blocks), dim3(threads), 0, s, w, w_ref, (u64)n, &ws->ext64, chunk_maxexp, part_max);
        return;
    }
#define LC_HIST(...) hipLaunchKernelGGL((k_hist<__VA_ARGS__>), dim3((u32)blocks), dim3(threads), 0, s, w, w_ref, (u64)n, ws, chunk_maxexp, batch_max, keys)
    // 2-byte elements that start between two dwords: a vector there takes longer than on a dword (2,048 chunks 31 us of this sweep and
    // 24), and as long as both arrays fit the last-level cache, 256 MB, element by element is faster.  By vectors / by elements, us the
    // call, bf16 unchanged; heavy tails; symbols of one scale: 520 chunks 36.1 / 34.8, 41.9 / 40.7, 52.5 / 52.0; 2,048 55.7 / 48.6, 65.2 /
    // 58.3, 93.4 / 85.3; 4,096 83.1 / 72.9, 99.8 / 88.9, 154.5 / 141.8; 6,000 109.1 / 114.2, 114.8 / 121.3, 212.0 / 195.3; 16,384 251.0 /
    // 262.3, 261.6 / 276.6, 523.9 / 512.1.
    const bool halves = ((reinterpret_cast<uintptr_t>(w) | reinterpret_cast<uintptr_t>(w_ref)) & 2) != 0 &&
                        num_chunks_of(n) <= 16 * (u64)tune.num_cu;
    if (dtype == kBF16) { if (halves) LC_HIST(kBF16, false, true); else LC_HIST(kBF16); }
    else if (dtype == kF16) { if (halves) LC_HIST(kF16, false, true); else LC_HIST(kF16); }
    else if (keys.exp) LC_HIST(kF32, true);
    else LC_HIST(kF32);
#undef LC_HIST
}

// Whether sweep 2 takes its chunks from a list of those to read.  Writing the list is work for the table's kernel, and taking
// chunks from it one more wait on memory for every workgroup; without it a workgroup finds out by itself that its chunk holds
// merged elements only, a wait each before it makes room for the next.  Without / with a list, whole calls, us: 2^20 fp32
// 39.3 / 40.8; 2^24 dense 87 / 88, sparse 64 / 59; 2^25 dense 128 / 134, sparse 90 / 81 (before: 86), 3 * 2^24 sparse 117 /
// 105.  2-byte elements, whose chunks take half the time to read: 2^23 dense 55.6 / 56.9, sparse 43.8 / 41.0; 2^24 dense
// 69.9 / 71.6, sparse 53.4 / 45.1.  A batched call has a kernel of its own for the list: 1,000 chunks 94 / 96, 2,000 140 / 142.
static bool needs_list(u64 nchunks, int per_cu, const Tuning& tune) { return nchunks > (u64)tune.num_cu * per_cu; }
bool pack_needs_list(uint64_t n, int dtype, const Tuning& tune) {
    return dtype == kF64 || needs_list(num_chunks_of(n), dtype == kF32 ? tune.unlisted_per_cu : tune.unlisted_per_cu / 2, tune);
}

void launch_pack_keys(const void* w, const void* w_ref, uint64_t n, Workspace* ws, uint32_t* chunk_bits, uint32_t* group_words,
                      const uint32_t* chunk_maxexp, const uint32_t* chunk_list, KeyPlanes keys, uint32_t* prov, uint32_t slot_words,
                      hipStream_t s) {
    const u64 nchunks = num_chunks_of(n);
    if (nchunks == 0) return;
    hipLaunchKernelGGL(k_pack_keys, dim3((u32)nchunks), dim3(kWgThreads), 0, s, w, w_ref, (u64)n, ws, chunk_bits, group_words, chunk_maxexp, chunk_list,
                       keys, prov, slot_words);
}

void launch_encode_one(const void* w, const void* w_ref, uint64_t n, int nbits, int dtype, uint8_t* out, Workspace* ws, uint32_t* record_words,
                       TableCache* cache, Result* host_result, uint64_t (&met)[kMeetLines], int looks, hipStream_t s) {
    const u32 nchunks = (u32)num_chunks_of(n);
    OneArgs a = {w, w_ref, (u64)n, out, ws, record_words, cache, host_result, {}, nchunks, 0, 0, nbits};
    set_goals(a, nchunks, met, looks);
    if (dtype == kBF16) hipLaunchKernelGGL(k_encode_one<kBF16>, dim3(nchunks), dim3(kWgThreads), 0, s, a);
    else if (dtype == kF16) hipLaunchKernelGGL(k_encode_one<kF16>, dim3(nchunks), dim3(kWgThreads), 0, s, a);
    else hipLaunchKernelGGL(k_encode_one<kF32>, dim3(nchunks), dim3(kWgThreads), 0, s, a);
}

// chunk_list: where to list the chunks sweep 2 has to read (chunk_maxexp then holds what k_hist recorded), or null
void launch_table(Workspace* ws, uint64_t n, int nbits, int dtype, uint32_t* group_words, const uint32_t* chunk_maxexp,
                  uint32_t* chunk_list, hipStream_t s) {
    const dim3 wg(chunk_list || dtype == kF64 ? 1024 : table_threads<8>());
    const u32 ngroups = (u32)((num_chunks_of(n) + 63) / 64);
    if (dtype == kF64) hipLaunchKernelGGL(k_table<11>, dim3(1), wg, 0, s, ws, &ws->ext64, (u64)n, nbits, group_words, ngroups, chunk_maxexp, chunk_list);
    else hipLaunchKernelGGL(k_table<8>, dim3(1), wg, 0, s, ws, &ws->ext64, (u64)n, nbits, group_words, ngroups, chunk_maxexp, chunk_list);
}

// Single-wave workgroups for a sweep over `nchunks` chunks dealt round-robin, at most `cap`: the largest count that
// gives every wavefront the same number of chunks (to within one), so that none is left with a turn of its own.
static u32 even_waves(u64 nchunks, u64 cap) {
    if (nchunks <= cap) return (u32)nchunks;
    const u64 turns = (nchunks + cap - 1) / cap;
    return (u32)((nchunks + turns - 1) / turns);
}

void launch_spec_table(Workspace* ws, const TableCache* cache, uint64_t n, int nbits, int dtype, uint32_t* group_words, hipStream_t s) {
    const u32 ngroups = (u32)((num_chunks_of(n) + 63) / 64);
    if (dtype == kF64) hipLaunchKernelGGL(k_spec_table<11>, dim3(1), dim3(64), 0, s, ws, &ws->ext64, cache, nbits, group_words, ngroups);
    else hipLaunchKernelGGL(k_spec_table<8>, dim3(1), dim3(64), 0, s, ws, (Ext64*)nullptr, cache, nbits, group_words, ngroups);
}

void launch_spec_sweep(const void* w, const void* w_ref, uint64_t n, int dtype, Workspace* ws, uint32_t* chunk_bits,
                       uint32_t* group_words, uint32_t* prov, uint32_t slot_words, const Tuning& tune, hipStream_t s) {
    const u64 nchunks = num_chunks_of(n);
    if (nchunks == 0) return;
    const u32 blocks = even_waves(nchunks, (u64)tune.num_cu * tune.spec_waves_per_cu);
    const dim3 grid(blocks), wg(64);
    if (dtype == kBF16) hipLaunchKernelGGL(k_spec_sweep<kBF16>, grid, wg, 0, s, w, w_ref, (u64)n, ws, chunk_bits, group_words, prov, slot_words, (u32)nchunks);
    else if (dtype == kF16) hipLaunchKernelGGL(k_spec_sweep<kF16>, grid, wg, 0, s, w, w_ref, (u64)n, ws, chunk_bits, group_words, prov, slot_words, (u32)nchunks);
    else hipLaunchKernelGGL(k_spec_sweep<kF32>, grid, wg, 0, s, w, w_ref, (u64)n, ws, chunk_bits, group_words, prov, slot_words, (u32)nchunks);
}

// chunk_maxexp, chunk_list: what k_hist recorded and k_table listed for this vector, or both null
void launch_pack(const void* w, const void* w_ref, uint64_t n, int dtype, Workspace* ws, uint32_t* chunk_bits,
                 uint32_t* group_words, const uint32_t* chunk_maxexp, const uint32_t* chunk_list, const uint8_t* batch_max,
                 uint32_t* prov, uint32_t slot_words, const Tuning& tune, hipStream_t s) {
    const u64 nchunks = num_chunks_of(n);
    if (nchunks == 0) return;
    // (a short call's chunks were not listed: see pack_needs_list)
    const u32* list = pack_needs_list(n, dtype, tune) ? chunk_list : nullptr;
    const u32* maxexp = chunk_list ? chunk_maxexp : nullptr;
    const dim3 wg(kWgThreads);
#define LC_PACK(DT, STAY, GRID) hipLaunchKernelGGL((k_pack<DT, STAY>), dim3((u32)(GRID)), wg, 0, s, w, w_ref, (u64)n, ws, chunk_bits, group_words, maxexp, list, batch_max, prov, slot_words, (u32)nchunks)
    if (dtype == kF64) {
        hipLaunchKernelGGL(k_pack64, dim3(even_waves(nchunks, (u64)tune.num_cu * tune.pack_waves_per_cu)), dim3(64), 0, s, w, w_ref, (u64)n, ws, &ws->ext64, chunk_bits, group_words, chunk_maxexp, chunk_list, batch_max, prov, slot_words, (u32)nchunks);
    } else if (chunk_list) {
        // a workgroup per chunk
        if (dtype == kBF16) LC_PACK(kBF16, false, nchunks);
        else if (dtype == kF16) LC_PACK(kF16, false, nchunks);
        else LC_PACK(kF32, false, nchunks);
    } else {
        // behind a speculative sweep there is mostly nothing to do, and starting 21,657 workgroups for that took 10 us instead
        // of 4: as many as start in that time, which take several chunks each when there is (354.8 M elements, coded anew /
        // confirmed: 4 per unit 1027 / 604 us, 8 1012 / 603, 16 1027 / 605, 64 1018 / 611; 2^26 236 / 154, 233 / 154)
        const u64 most = (u64)tune.num_cu * 8, grid = nchunks < most ? nchunks : most;
        if (dtype == kBF16) LC_PACK(kBF16, true, grid);
        else if (dtype == kF16) LC_PACK(kF16, true, grid);
        else LC_PACK(kF32, true, grid);
    }
#undef LC_PACK
}

// The placement of all chunks and, in the same launch, the header and the call's outcome (result: mapped host memory;
// cache: lc_encode_cached's, or null; staged: the extremes come from sweep 1's per-bucket record).
void launch_place(uint8_t* out, Workspace* ws, const uint32_t* chunk_bits, const uint32_t* group_words,
                  const uint32_t* prov, uint32_t slot_words, uint64_t n, uint32_t* chunk_maxexp, Result* host_result,
                  TableCache* cache, int nbits, int dtype, bool staged, hipStream_t s) {
    const u64 nchunks = num_chunks_of(n);
    const u32 blocks = (u32)((nchunks + 3) / 4) + 1;             // + the workgroup that writes the header
    const FinalizeArgs fin = {host_result, cache, (u64)n, nbits, (u32)dtype, staged ? 1 : 0};
    // (up to 1024 workgroups are resident together on this chip even with the larger windows)
    if (blocks <= 1024u) hipLaunchKernelGGL(k_place<kPlaceWordsFew>, dim3(blocks), dim3(256), 0, s, out, ws, chunk_bits, group_words, prov,
                                                slot_words, (u32)nchunks, chunk_maxexp, fin);
    else hipLaunchKernelGGL(k_place<kPlaceWords>, dim3(blocks), dim3(256), 0, s, out, ws, chunk_bits, group_words, prov,
                            slot_words, (u32)nchunks, chunk_maxexp, fin);
}

void launch_batch_encode(const BatchArgs& args, const Tuning& tune, hipStream_t s) {
    BatchArgs a = args;
    a.listed = needs_list(a.total_chunks, tune.batch_unlisted_per_cu, tune) ? 1 : 0;
    hipLaunchKernelGGL(kb_setup, dim3(a.count), dim3(256), 0, s, a);
    if (a.total_chunks) {
        // A workgroup per chunk as the dispatcher hands them out, or two per compute unit that stay: a tensor's workgroups hand in
        // some 40 counts each to the same few lines of memory, and few streams of long bursts read faster.  Whole calls, us, per
        // chunk / staying: fp32 2^24.6 115 / 117, 2^25 131 / 137, 2^26 233 / 215, 138 M 284 / 249, 2^27 471 / 435; bf16 2^25 105 /
        // 115, 2^26 158 / 165, 2^27 270 / 258.  (1, 3 and 4 per unit 458, 467, 443 for the last fp32 one)
        // Up to half a chunk on average, the form for few rows.
        const bool stay = a.total_chunks >= (u32)tune.num_cu * (a.dtype == kF32 ? 12u : 24u);
        const u32 most = 2 * (u32)tune.num_cu, run = stay ? (a.total_chunks + most - 1) / most : 1;
        const dim3 grid((a.total_chunks + run - 1) / run), wg(kWgThreads);
#define LC_HIST(DT) do { if (stay) hipLaunchKernelGGL((kb_hist<DT, true>), grid, wg, 0, s, a, run); \
                         else if (a.mean <= 4 * kWgRows * kRowElems) hipLaunchKernelGGL((kb_hist<DT, false, true>), grid, wg, 0, s, a, run); \
                         else hipLaunchKernelGGL((kb_hist<DT, false>), grid, wg, 0, s, a, run); } while (0)
        if (a.dtype == kBF16) LC_HIST(kBF16);
        else if (a.dtype == kF16) LC_HIST(kF16);
        else LC_HIST(kF32);
#undef LC_HIST
    }
    hipLaunchKernelGGL(kb_table, dim3(a.count), dim3(table_threads<8>()), 0, s, a);
    if (a.total_chunks) {
        if (a.listed) hipLaunchKernelGGL(kb_list, dim3((a.total_chunks + 255) / 256), dim3(256), 0, s, a);
        const dim3 grid(a.total_chunks), wg(kWgThreads);
        if (a.dtype == kBF16) hipLaunchKernelGGL(kb_pack<kBF16>, grid, wg, 0, s, a);
        else if (a.dtype == kF16) hipLaunchKernelGGL(kb_pack<kF16>, grid, wg, 0, s, a);
        else hipLaunchKernelGGL(kb_pack<kF32>, grid, wg, 0, s, a);
    }
    hipLaunchKernelGGL(kb_place, dim3(a.count + (a.total_chunks + 3) / 4), dim3(256), 0, s, a);
}

}  // namespace lc
