// Decode kernels of the LC-Checkpoint compress / restore path for gfx950 (wave64): restore by
// accumulation (Algorithm 1 line 7; Section 3, C1).
//
// lc_decode:        k_dec_check -> k_decode (gated on the check's verdict, no host round trip between); a short vector: k_decode_one
// lc_decode_many:   k_dec_check (all blobs) -> k_decode_fused<T> or k_decode_pairs<T> per sweep; of a short vector mostly k_decode_one
// lc_decode_batch:  kb_dec_tables -> kb_dec_chunks -> kb_decode
#include "lc_device.h"
#include <type_traits>

namespace lc {

// ----------------------------------------------------------------------------- k_dec_check
// Tables of one blob while its workgroup builds them.
struct DecBuild {
    u32 len[kMaxSym], code[kMaxSym], max_len;
    uint8_t one[1u << kMultiBits];            // over the next 10 bits: symbol | len << 4 of the first code (see dec_build_luts)
};

// The same by the first wavefront of a workgroup, left in D.info for the sweep and in B for dec_build_luts.
__device__ __forceinline__ bool dec_symbol_table(const u32* hdr, u64 n, u32 nchunks, u64 area, u64 tw, DecSet& D, DecBuild& B) {
    const u32 lane = lane_id();
    DecSymbol sy;
    const bool ok = dec_symbols(hdr, n, nchunks, tw, &sy);
    const u32 max_len = wave_max_u32(sy.len);
    if (lane < kMaxSym) {
        B.len[lane] = sy.len; B.code[lane] = sy.code;
        D.info.rep_bits[lane] = sy.rep; D.info.rep_hi[lane] = sy.rep_hi;
        D.info.len[lane] = sy.len; D.info.code[lane] = sy.code;
    }
    if (lane == 0) { B.max_len = max_len; D.info.K = hdr[5]; D.info.max_len = max_len; D.info.area = area; D.info.total_words = tw; }
    return ok;
}

// By a workgroup of 256 threads, from what dec_symbol_table left in B; D.lut1 is the table of single symbols over 7 bits, for
// the fused restore.
__device__ __forceinline__ void dec_build_luts(DecSet& D, DecBuild& B, u32 K, u32 t) {
    const u32 lane = t & (kW - 1);
    const u32 len = lane < kMaxSym ? B.len[lane] : 0u, code = lane < kMaxSym ? B.code[lane] : 0u;
    // (a prefix that starts no code: nothing is ever taken off again, and the lane falls short of its stated length)
    dec_build_multi<256>(D.multi, B.one, nullptr, (K * 0x111111u) | (kMultiSyms << 28), len, code, t);
    const u32 M = wave_max_u32(len), P1 = M < kDecLut1Bits ? M : kDecLut1Bits;
    if (t < (1u << P1)) {
        const u32 f = B.one[t << (kMultiBits - P1)];
        D.lut1[t] = f == kOneNone ? (uint8_t)K : (f >> 4) > P1 ? (uint8_t)0xFF : (uint8_t)f;
    }
}

// One chunk's place in the offset table against the lane lengths of its record, by one wavefront.
__device__ __forceinline__ bool dec_chunk_ok(const uint8_t* blob, u64 area, u64 tw, u32 nchunks, u32 c) {
    const u32* off_tab = reinterpret_cast<const u32*>(blob + kHeaderBytes);
    const u64 o0 = off_tab[c], o1 = off_tab[c + 1];
    bool ok = o0 <= o1 && o1 <= tw && o1 - o0 >= kLaneBitsWords && (c > 0 || o0 == 0) && (c + 1 < nchunks || o1 == tw);
    if (ok) {
        const u32 lb = reinterpret_cast<const uint16_t*>(blob + area + 4 * o0)[lane_id()];
        const u32 sum = wave_sum32(lb);
        ok = (o1 - o0 == kLaneBitsWords + ((sum + 31) >> 5)) && sum > 0 && !__any(lb > kR * kV * 15);
    }
    return ok;
}

// The same for chunks c0 .. c0 + 3 at once (their loads in flight together); false if any of those below nchunks fails.
__device__ __forceinline__ bool dec_chunks_ok4(const uint8_t* blob, u64 area, u64 tw, u32 nchunks, u32 c0) {
    const u32* off_tab = reinterpret_cast<const u32*>(blob + kHeaderBytes);
    const u32 lane = lane_id();
    u64 o[5];
#pragma unroll
    for (u32 k = 0; k < 5; ++k) o[k] = c0 + k <= nchunks ? off_tab[c0 + k] : 0;
    bool ok[4];
    u32 lb[4];
#pragma unroll
    for (u32 k = 0; k < 4; ++k) {
        const u32 c = c0 + k;
        ok[k] = c < nchunks && o[k] <= o[k + 1] && o[k + 1] <= tw && o[k + 1] - o[k] >= kLaneBitsWords && (c > 0 || o[k] == 0) &&
                (c + 1 < nchunks || o[k + 1] == tw);
        lb[k] = ok[k] ? reinterpret_cast<const uint16_t*>(blob + area + 4 * o[k])[lane] : 0u;
    }
    bool all = true;
#pragma unroll
    for (u32 k = 0; k < 4; ++k) {
        if (c0 + k >= nchunks) continue;
        const u32 sum = wave_sum32(lb[k]);
        all = all && ok[k] && (o[k + 1] - o[k] == kLaneBitsWords + ((sum + 31) >> 5)) && sum > 0 && !__any(lb[k] > kR * kV * 15);
    }
    return all;
}

// Everything lc_decode verifies before w_ref is touched, in one launch.  Every workgroup
// re-reads the header and does the cheap sanity checks that keep its own reads in bounds;
// workgroup 0 additionally validates the symbol table, rebuilds the canonical codes and the
// look-up table; each wavefront checks one chunk: the offset table must be the running sum
// of the record sizes that the lane lengths imply, from 0 to the blob's stated size.
// Errors are raised with atomicMax on a word tagged with the call's epoch, so the word
// never needs clearing.
// PER: chunks per wavefront, 1 or 4 (4 when one chunk each would take many rounds of workgroups: several blobs, or a long one)
template <int PER>
__global__ __launch_bounds__(256) void k_dec_check(BlobList blobs, u32 first, u64 n, u64 max_total, Workspace* ws,
                                                   u32 nchunks, u64 epoch, HostResult* host, u32 dtype) {
    const u32 set = first + blockIdx.y, host_slot = set;     // one grid row per blob
    const uint8_t* blob = blobs.p[set];
    __shared__ u32 hdr[kHeaderBytes / 4];
    __shared__ u32 s_ok;
    __shared__ DecBuild B;
    const u32 t = threadIdx.x, lane = lane_id();
    if (t < kHeaderBytes / 4) hdr[t] = reinterpret_cast<const u32*>(blob)[t];
    __syncthreads();
    const u64 hn = hdr[2] | ((u64)hdr[3] << 32), total = hdr[10] | ((u64)hdr[11] << 32);
    const u64 area = chunk_area_of(nchunks);
    const bool head_ok = hdr[0] == 0x3142434Cu && hdr[1] == (1u | (kHeaderBytes << 16)) && hdr[12] == 0 &&
                         hn == n && hdr[15] == dtype && hdr[9] == nchunks && total >= area && total <= max_total &&
                         ((total - area) & 3) == 0;
    if (!head_ok) {
        if (blockIdx.x == 0 && t == 0) {
            const bool n_mismatch = hdr[0] == 0x3142434Cu && hdr[1] == (1u | (kHeaderBytes << 16)) && hdr[12] == 0 &&
                                    (hn != n || hdr[15] != dtype);       // a sound blob for another vector or element type
            raise_status(ws, host, epoch, n_mismatch ? 1u : 4u);
            host->bytes[host_slot] = 0; host->max_len[host_slot] = 0;
        }
        return;
    }
    const u64 tw = (total - area) / 4;
    // ---- one chunk, or four, per wavefront
    const u32 c0 = (blockIdx.x * 4 + (t >> 6)) * PER;
    if (c0 < nchunks) {
        const bool ok = PER == 4 ? dec_chunks_ok4(blob, area, tw, nchunks, c0) : dec_chunk_ok(blob, area, tw, nchunks, c0);
        if (!ok && lane == 0) raise_status(ws, host, epoch, 4u);
    }
    if (blockIdx.x != 0) return;
    // ---- workgroup 0: symbol table, codes, look-up table
    DecSet& D = ws->dec_set[set];
    if (t < kW) {
        const bool ok = dec_symbol_table(hdr, n, nchunks, area, tw, D, B);
        if (t == 0) {
            if (!ok) raise_status(ws, host, epoch, 4u);
            host->bytes[host_slot] = total; host->max_len[host_slot] = B.max_len; host->kept[host_slot] = hdr[5];
            s_ok = ok;
        }
    }
    __syncthreads();
    if (!s_ok) return;
    dec_build_luts(D, B, hdr[5], t);
}

// ----------------------------------------------------------------------------- k_decode
// Algorithm 1 line 7: one wavefront per chunk, lane l decoding its own string.  The chunk's payload is first copied to LDS
// with coalesced 16-byte loads, so the lanes' word-by-word refills never go to memory.
//
// Decoding is a serial chain per lane (the next code starts where this one ends), and what it costs is not bytes but the
// steps of that chain: at one symbol per look-up, an LDS round trip and some 16 instructions per symbol.  Here a look-up
// yields all the whole codes that the next 10 bits hold, up to 6 (3 on average with codes of 3 bits, 5 with codes of 1.7),
// and the lanes, which then advance at different rates, leave their symbols (4 bits each) in a ring in LDS: 8 words of 8
// symbols per lane, word k of lane l at [64 (k mod 8) + l], so that no two lanes ever meet in a bank.  A lane that is
// ahead goes on until its ring is full; the slowest decides when the next 8 rows are complete.  Those rows of w_ref, which
// were asked for 8 rows earlier, then take their representatives in a second loop that has no chain at all.
// One symbol per look-up against this (whole calls, which also have a faster check): 2^20 fp32 elements 47.7 -> 35.8 us,
// 161 tensors of 25.6 M 131 -> 88 us, 2^27 bf16 138 -> 129 us; the dense slice of 2^28 fp32, which moves 2.25 GB at what a
// bare read-and-write sweep in this walk reaches (5.5 TB/s), 437 -> 421 us.
// The merged symbol adds -0.0, which leaves every fp32 pattern unchanged, and a row in which no lane decoded a kept symbol
// is not written back at all.
// LDS room for one chunk's payload.  A longer one is read from memory, lane by lane, 2-3 times as slow for that chunk, so a
// launch takes as much as leaves room for the workgroups that will share a compute unit: (32 chunks of 7.5 bits per element in
// 2^25: 98 us with 3072 words, 81 with 4224; one in 2^23: 82 and, with room for any, 74)
constexpr u32 kPayWords = 2048;      // three: 4 bits per element on average
constexpr u32 kPayWordsTwo = 4224;   // two: 8 bits
constexpr u32 kPayWordsVerify = 3040;               // three of the verifying sweep, which has no ring (2^28 dense elements 95 us, 119 with two)
constexpr u32 kPayWordsOne = kChunk * 15 / 32 + 4;  // one: 15 bits, the longest payload there is, wherever it starts in a vector
constexpr u32 kRingWords = 8;        // words of 8 symbols that a lane may be ahead of the rows being restored
constexpr u32 kGroupRows = 8;        // rows restored at a time: 32 symbols, 4 words of the ring per lane

// What a wavefront keeps of a blob's code in registers, the same in every lane.
struct CodeLens {
    u64 nibbles;                      // the length of symbol j at bits 4 j
    u32 sparse;                       // the merged symbol's length if it is below every other's, else 0
    __device__ __forceinline__ u32 of(u32 sy) const { return (u32)(nibbles >> (4 * sy)) & 15u; }
    // by a whole wavefront, lane j holding the length of symbol j (0 in lanes without one)
    __device__ __forceinline__ void set(u32 len, u32 K) {
        const u32 lane = lane_id(), mine = lane < kMaxSym ? len << (4 * (lane & 7)) : 0u;
        const u32 lo = wave_sum32(lane < 8 ? mine : 0u), hi = wave_sum32(lane < 8 ? 0u : mine);
        nibbles = ((u64)hi << 32) | lo;
        const u32 merged = read_lane(len, K);
        sparse = __any(lane < K && len != 0 && len <= merged) ? 0u : merged;
    }
};

// `raise(code)` reports a lane string that does not decode to its stated length.
// LONG: the blob has codes of more than 10 bits.
// VERIFY: the lane strings are only decoded and measured against their stated lengths; w_ref is not touched (nor read).
// ring: this wavefront's kRingWords * 64 words of LDS.
template <bool FAST, bool LONG, bool STAGED, int DT, bool VERIFY, typename LDS, typename Raise>
__device__ __forceinline__ void decode_rows(const u32* words, u32 nwords, u32 first_bit, u32 lane_bits,
                                            void* __restrict__ w_ref, u64 n, u32 c,
                                            const LDS& L, u32* ring, u32 K, const CodeLens& lens, bool ahead, Raise& raise) {
    typedef typename Val<DT>::type val_t;
    const u32 lane = lane_id();
    BitReader<STAGED> br;
    br.start(words, nwords, first_bit);
    const u32 wi0 = br.wi, avail0 = br.avail;
    const u64 base = (u64)c * kChunk;
    // Places in a lane's string of symbols are counted in bits of the ring, 4 to a symbol.
    constexpr int kGroupQ = kGroupRows * kV * 4, kRingQ = kRingWords * 32, kStepQ = kMultiSyms * 4;
    static_assert(kRingQ == 2 * kGroupQ && kStepQ < 32, "a step fills at most one word; the ring holds two groups");
    int limit = kR * kV * 4;                             // the end of this lane's string
    if (!FAST) {
        const u32 left = n - base < kChunk ? (u32)(n - base) : kChunk, tail = left % kRowElems;
        const u32 mine = tail > lane * kV ? min(tail - lane * kV, kV) : 0u;
        limit = (int)((left / kRowElems * kV + mine) * 4);
    }
    int q = 0;                                           // symbols so far, and
    u32 acc = 0;                                         // those of the word of the ring that is being filled
    u32* mine = ring + lane;
    auto append = [&](u32 e) {
        const u64 s = (u64)(e & 0xFFFFFFu) << (q & 31);
        acc |= (u32)s;
        if (!VERIFY) mine[((q >> 5) & (kRingWords - 1)) * kW] = acc;       // (a partly filled word is written again by the next step)
        const int qn = q + (int)((e >> 28) << 2);
        if ((qn ^ q) & 32) acc = (u32)(s >> 32);
        q = qn;
        br.drop((e >> 24) & 15u);
    };
    // all the codes of the next 10 bits, by the lanes that have not come to `cap` (33 valid bits take three such steps,
    // two if one of them may be a code of up to 15 bits)
    auto step = [&](int cap) {
        u32 e = L.multi[(u32)(br.win >> (64 - kMultiBits))];
        if (LONG && __any(q < cap && e == 0)) { if (e == 0) e = decode_long(L, br.win); }
        append(q < cap ? e : 0u);
    };
    // the next code alone, by the lanes that have not come to `end`
    auto one = [&](int end) {
        u32 e = L.multi[(u32)(br.win >> (64 - kMultiBits))];
        if (LONG && __any(e == 0)) { if (e == 0) e = decode_long(L, br.win); }
        const u32 sy = e & 15u, len = (e & 0x0F000000u) ? lens.of(sy) : 0u;       // (length 0: a prefix that starts no code)
        append(q < end ? (sy | (len << 24) | (1u << 28)) : 0u);
    };
    // the symbols of group g, complete in the ring
    const int stop = limit - kStepQ + 4;                 // from here on a step could pass the end of the string
    auto symbols = [&](u32 g) {
        const int end = min((int)(g + 1) * kGroupQ, limit), many = min(end, stop);
        const int cap = min((int)g * kGroupQ + kRingQ - kStepQ, stop);         // (no word of this group is overwritten)
        while (__any(q < many)) {
            step(cap);
            step(cap);
            if (!LONG) step(cap);
            br.refill();
        }
        if (!FAST || g + 1 == kR / kGroupRows)
            while (__any(q < end)) { one(end); br.refill(); }
        // (a ragged chunk: the step that finished a lane's string may have gone over into a word that no step has written)
        if (!FAST && !VERIFY) mine[((q >> 5) & (kRingWords - 1)) * kW] = acc;
    };
    auto row_at = [&](u32 r) { return base + (u64)r * kRowElems + lane * kV; };
    // the 4 symbols of row k of group g, as the low 16 bits
    auto row_syms = [&](u32 g, u32 k) { return mine[((g * (kGroupRows / 2) + k / 2) & (kRingWords - 1)) * kW] >> (16 * (k & 1)); };
    auto any_kept = [&](u32 syms) { return __any(((syms ^ (K * 0x1111u)) & 0xFFFFu) != 0); };
    auto add_row = [&](u32 syms, val_t (&x)[4]) {
#pragma unroll
        for (int v = 0; v < 4; ++v) x[v] = add_rn(x[v], L.template rep_of<DT>((syms >> (4 * v)) & 15u));
    };
    auto check = [&]() {
        const u32 used = avail0 + 32 * (br.wi - wi0) - br.avail;
        if (__any(used != lane_bits) && lane == 0) raise(4u);
    };
    br.refill();
    if constexpr (VERIFY) {
        for (u32 g = 0; g < kR / kGroupRows && (FAST || base + (u64)g * kGroupRows * kRowElems < n); ++g) symbols(g);
    } else if constexpr (FAST) {
        typedef typename Raw<DT>::type raw_t;
        // (binary64: plain loads, since a lane's 32 bytes are two loads from the same lines: marked non-temporal, 2^24
        // elements 76 us and 62 so, 2^26 267 and 243, layers of 2^25 125 and 98)
        auto fetch = [&](raw_t (&X)[kGroupRows], u32 g) {
#pragma unroll
            for (u32 k = 0; k < kGroupRows; ++k) X[k] = load_raw_any<DT, DT != kF64>(w_ref, row_at(g * kGroupRows + k));
        };
        auto restore = [&](const raw_t (&X)[kGroupRows], u32 g) {
#pragma unroll
            for (u32 k = 0; k < kGroupRows; ++k) {
                const u32 syms = row_syms(g, k);
                if (!any_kept(syms)) continue;
                val_t x[4];
                if constexpr (DT == kF64) unpack64(X[k], x); else unpack<DT>(X[k], x);
                add_row(syms, x);
                store4_any<DT>(w_ref, row_at(g * kGroupRows + k), x);
            }
        };
        // (ahead: the next group's rows are asked for before this one is decoded; else only its own, and the wavefronts that
        // share a SIMD cover each other's waits.  binary64 rows are 2 KiB: ahead, 2^24 elements 62 us against 64, layers of 2^25
        // 98 against 96, of 2^26 210 against 200)
        // Off alignment the same rows: the hardware takes vectors at any address.  Against guarded loads and stores of single
        // elements and a look-up for codes of any length, 2^27 elements in layers 350 -> 187 us (fp32; aligned 180) and
        // 462 -> 175 (bf16; 156), a batch of 32 layers of 2^20 96 -> 87 and 135 -> 93; binary64 in layers 2^25 115 -> 99, of one
        // scale 2^24 83 -> 62, 2^25 129 -> 132, 2^26 250 -> 244.
        if (DT != kF64 || ahead) {
            raw_t A[kGroupRows], B[kGroupRows];
            fetch(A, 0);
            for (u32 g = 0; g < kR / kGroupRows; g += 2) {
                fetch(B, g + 1);
                symbols(g);
                restore(A, g);
                if (g + 2 < kR / kGroupRows) fetch(A, g + 2);
                symbols(g + 1);
                restore(B, g + 1);
            }
        } else {
            for (u32 g = 0; g < kR / kGroupRows; ++g) {
                raw_t A[kGroupRows];
                fetch(A, g);
                symbols(g);
                restore(A, g);
            }
        }
    } else {
        // A ragged chunk (the vector's last chunk is one wavefront's work from start to end, so its memory round trips
        // count): rows that lie wholly inside the array as vectors, the rest element by element.
        for (u32 g = 0; g < kR / kGroupRows && base + (u64)g * kGroupRows * kRowElems < n; ++g) {
            val_t x[kGroupRows][4];
            auto fetch = [&](u32 k) {
                const u32 r = g * kGroupRows + k;
                if (base + (u64)(r + 1) * kRowElems <= n) load_row_any<DT, DT != kF64>(w_ref, row_at(r), x[k]);
                else load_row_v<DT>(w_ref, row_at(r), n, x[k]);
            };
#pragma unroll
            for (u32 k = 0; k < kGroupRows; ++k) fetch(k);               // on their way while the symbols are decoded
            symbols(g);
#pragma unroll
            for (u32 k = 0; k < kGroupRows; ++k) {
                const u32 r = g * kGroupRows + k, syms = row_syms(g, k);
                if (base + (u64)(r + 1) * kRowElems <= n) {
                    if (!any_kept(syms)) continue;
                    add_row(syms, x[k]);
                    store4_any<DT>(w_ref, row_at(r), x[k]);
                } else {
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const u32 sy = (syms >> (4 * v)) & 15u;
                        if (row_at(r) + v < n && sy != K) store_one_v<DT>(w_ref, row_at(r) + v, add_rn(x[k][v], L.template rep_of<DT>(sy)));
                    }
                }
            }
        }
    }
    check();
}

// A chunk of few kept symbols (the caller has seen that from its size), ragged or not: a lane goes from one to the next.  Its
// string is runs of the merged symbol's code, all zero bits and shorter than any other, which the leading zeros of the window
// count up to 32 bits at a time; only the symbols between them are looked up.  They are noted in the lane's column of `noted`
// (kRingWords of them) and added to their elements when some column is full, the elements of all lanes in flight together;
// nothing else of w_ref is read or written.
// Against the rows around the kept symbols restored, with a look-up for each of a row's symbols: 2^20 fp32 elements of one
// scale at 2 bits 61 -> 28 us (52 when symbol and length were one look-up), 2^26 of a drift 137 -> 38 us (93), 138 M of a
// sparse update 37 -> 29 us (40).
template <int DT, typename LDS, typename Raise>
__device__ __forceinline__ void decode_sparse(const u32* words, u32 nwords, u32 first_bit, u32 lane_bits, u32 lane_elems,
                                              void* __restrict__ w_ref, u64 base, const LDS& L, u32* noted, u32 K,
                                              const CodeLens& lens, Raise& raise) {
    const u32 lane = lane_id();
    BitReader<true> br;
    br.start(words, nwords, first_bit);
    const u32 wi0 = br.wi, avail0 = br.avail;
    const u32 m = lens.sparse, inv = 65536u / m + 1;               // (z inv >> 16 = z / m for z <= 32, m <= 15)
    u32* mine = noted + lane;
    u32 pos = 0, count = 0;
    auto add_noted = [&]() {
        u32 e[kRingWords];
        typename Val<DT>::type x[kRingWords];
        auto at = [&](u32 k) { const u32 p = e[k] >> 4; return base + (u64)((p / kV) * kRowElems + lane * kV + p % kV); };
#pragma unroll
        for (u32 k = 0; k < kRingWords; ++k) if (k < count) { e[k] = mine[k * kW]; x[k] = load_one_v<DT>(w_ref, at(k)); }
#pragma unroll
        for (u32 k = 0; k < kRingWords; ++k) if (k < count) store_one_v<DT>(w_ref, at(k), add_rn(x[k], L.template rep_of<DT>(e[k] & 15u)));
        count = 0;
    };
    br.refill();
    while (__any(pos < lane_elems)) {
        const u32 top = (u32)(br.win >> 32), zeros = top != 0 ? (u32)__builtin_clz(top) : 32u;
        const u32 run = min(zeros * inv >> 16, lane_elems - pos);
        pos += run;
        br.drop(run * m);
        br.refill();
        const bool kept = pos < lane_elems && (u32)(br.win >> (64 - m)) != 0;
        if (__any(kept)) {
            u32 e = L.multi[(u32)(br.win >> (64 - kMultiBits))];
            if (__any(kept && e == 0)) { if (e == 0) e = decode_long(L, br.win); }
            const u32 sy = e & 15u;
            if (kept) {
                mine[count * kW] = (pos << 4) | sy;
                count += sy != K ? 1u : 0u;                        // (K: a prefix that starts no code)
                ++pos;
                br.drop((e & 0x0F000000u) ? lens.of(sy) : 0u);
            }
            br.refill();
            if (__any(count == kRingWords)) add_noted();
        }
    }
    if (__any(count != 0)) add_noted();
    if (__any(avail0 + 32 * (br.wi - wi0) - br.avail != lane_bits) && lane == 0) raise(4u);
}

// zero_bits: what every lane length of a full chunk is when all its elements are the merged symbol and that
// symbol's code is all zero bits (the canonical first code), else 0.  Such a chunk with an all-zero payload
// decodes to the merged symbol throughout, exactly: it changes nothing and is left without reading w_ref.
__device__ __forceinline__ u32 zero_chunk_bits(u32 len_merged, u32 code_merged) {
    return (len_merged != 0 && code_merged == 0) ? kR * kV * len_merged : 0u;
}

// A chunk's record looked at where it lies, to tell whether it is such a chunk's: nothing is staged for it, and a wavefront
// that meets no other chunk never needs the blob's tables.  The loads of `start` are on their way while the chunk before is
// restored; o0, o1: the chunk's entries of the offset table.
struct QuietChunk {
    const u32* rec;
    u32 nwords, differs, x[8];                  // payload words in all (0: the chunk's size alone says that it is none); the first 512
    __device__ __forceinline__ void start(const uint8_t* __restrict__ blob, u64 area, u32 o0, u32 o1, u32 zero_bits, bool full) {
        nwords = o1 - o0 - kLaneBitsWords;
        if (!full || zero_bits == 0 || nwords != zero_bits * kW / 32) { nwords = 0; return; }
        rec = reinterpret_cast<const u32*>(blob + area + 4 * (u64)o0);
        differs = reinterpret_cast<const uint16_t*>(rec)[lane_id()];
#pragma unroll
        for (int k = 0; k < 8; ++k) x[k] = rec[kLaneBitsWords + lane_id() + k * kW];      // (nwords: a multiple of 512)
    }
    __device__ __forceinline__ bool holds(u32 zero_bits) {
        if (nwords == 0) return false;
        differs ^= zero_bits;
        for (u32 i = 0;;) {
#pragma unroll
            for (int k = 0; k < 8; ++k) differs |= x[k];
            i += 8 * kW;
            if (i >= nwords) break;
#pragma unroll
            for (int k = 0; k < 8; ++k) x[k] = rec[kLaneBitsWords + i + lane_id() + k * kW];
        }
        return !__any(differs != 0);
    }
};

// pay: this wavefront's LDS area of pay_words + 4 words for the chunk's payload; ring: its symbol ring
// fast: a full chunk; long_codes: the blob has codes of more than 10 bits; ahead: see decode_rows
template <int DT, bool VERIFY = false, typename LDS, typename Raise>
__device__ __forceinline__ void decode_chunk(const uint8_t* __restrict__ blob, void* __restrict__ w_ref, u64 n,
                                             u32 c, u32 o0, u32 o1, bool fast, bool long_codes, bool ahead, LDS& L, uint4* pay, u32 pay_words, u32* ring, u32 K,
                                             const CodeLens& lens, u64 area, Raise& raise) {
    // o0, o1: the chunk's entries c and c + 1 of the offset table (fetched by the caller, ahead of time)
    const u32 lane = lane_id();
    const uint8_t* rec = blob + area + 4 * (u64)o0;
    const u32 nwords = o1 - o0 - kLaneBitsWords;        // >= 1 (validated)
    const u32 lane_bits = reinterpret_cast<const uint16_t*>(rec)[lane];
    const u32* gw = reinterpret_cast<const u32*>(rec + 2 * kW);
    const u32 k0 = (u32)((reinterpret_cast<uintptr_t>(gw) >> 2) & 3);     // words between the 16-byte boundary and the payload
    const bool staged = nwords + k0 <= pay_words;
    if (staged) {
        // coalesced copy of [aligned start, payload end) to LDS; the bytes before the payload are the
        // record's own lane lengths, and the last vector is read word by word so no read passes the end
        const uint4* gv = reinterpret_cast<const uint4*>(gw - k0);
        const u32 nvec = (nwords + k0 + 3) >> 2;
        for (u32 i = lane; i < nvec; i += kW) {
            uint4 q;
            if (4 * i + 4 <= nwords + k0) q = gv[i];
            else {
                const u32* t = reinterpret_cast<const u32*>(gv + i);
                const u32 left = nwords + k0 - 4 * i;
                q.x = t[0]; q.y = left > 1 ? t[1] : 0; q.z = left > 2 ? t[2] : 0; q.w = 0;
            }
            pay[i] = q;
        }
    }
    const u32 incl = wave_incl_scan(lane_bits), o = incl - lane_bits;
    // Few kept symbols?  When the merged symbol's code is shorter than every other, each kept symbol costs at least
    // one bit more, so a chunk of at most kSparseSlack bits above (elements x merged length) holds at most that many;
    // and no lane may hold many of them, since the fullest sets the pace.
    const u64 left = n - (u64)c * kChunk;
    const u32 elems = left < kChunk ? (u32)left : kChunk, tail = elems % kRowElems;
    const u32 lane_elems = elems / kRowElems * kV + (tail > lane * kV ? min(tail - lane * kV, kV) : 0u);
    const bool sparse = !VERIFY && staged && lens.sparse != 0 && read_lane(incl, kW - 1) <= elems * lens.sparse + kSparseSlack &&
                        !__any(lane_bits > lane_elems * lens.sparse + kSparseLaneSlack);
    const u32* words = reinterpret_cast<const u32*>(pay) + k0;
    if constexpr (!VERIFY) {
        if (sparse) { decode_sparse<DT>(words, nwords, o, lane_bits, lane_elems, w_ref, (u64)c * kChunk, L, ring, K, lens, raise); return; }
    }
    if (staged) {
        if (!fast) decode_rows<false, true, true, DT, VERIFY>(words, nwords, o, lane_bits, w_ref, n, c, L, ring, K, lens, ahead, raise);
        else if (long_codes) decode_rows<true, true, true, DT, VERIFY>(words, nwords, o, lane_bits, w_ref, n, c, L, ring, K, lens, ahead, raise);
        else decode_rows<true, false, true, DT, VERIFY>(words, nwords, o, lane_bits, w_ref, n, c, L, ring, K, lens, ahead, raise);
    } else {
        if (!fast) decode_rows<false, true, false, DT, VERIFY>(gw, nwords, o, lane_bits, w_ref, n, c, L, ring, K, lens, ahead, raise);
        else if (long_codes) decode_rows<true, true, false, DT, VERIFY>(gw, nwords, o, lane_bits, w_ref, n, c, L, ring, K, lens, ahead, raise);
        else decode_rows<true, false, false, DT, VERIFY>(gw, nwords, o, lane_bits, w_ref, n, c, L, ring, K, lens, ahead, raise);
    }
}

// VERIFY: lc_verify's sweep (and the one lc_decode runs first when asked to): the same walk over the blob, decoding
// only; `w_ref` is not used.  ahead: rows are fetched a group ahead.
template <int DT, bool VERIFY = false>
__global__ __launch_bounds__(256, DT == kF64 ? 2 : 3) void k_decode(const uint8_t* __restrict__ blob, void* __restrict__ w_ref, u64 n,
                                                Workspace* ws, u32 nchunks, int ahead, u64 epoch, HostResult* host,
                                                u32 pay_words, u32 set) {
    __shared__ DecLds L;
    __shared__ u32 s_ring[VERIFY ? 1 : 4 * kRingWords * kW];
    extern __shared__ uint4 dec_pay[];                   // 4 areas of pay_words + 4 payload words, one per wavefront
    // What the check kernel left (the verdict and the blob's tables) is fetched in one go: a failed check leaves
    // tables that mean nothing, but reading them is harmless.  The blob itself is not: one that was refused may end
    // anywhere behind its header, so no load from it stands ahead of the verdict (nchunks comes from the caller's n).
    const u32 t = threadIdx.x;
    const DecSet& D = ws->dec_set[set];
    const u64 verdict = __hip_atomic_load(&ws->dec_status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    u32 M = D.info.max_len, K = D.info.K;
    u64 area = D.info.area;
    const u32 lane = t & (kW - 1);
    u32 sym_rep = 0, sym_rep_hi = 0, sym_len = 0, sym_code = 0;
    if (lane < kMaxSym) { sym_rep = D.info.rep_bits[lane]; sym_rep_hi = D.info.rep_hi[lane]; sym_len = D.info.len[lane]; sym_code = D.info.code[lane]; }
    const u32 wave = t >> 6, stride = gridDim.x * 4;
    const u32 first = blockIdx.x * 4 + wave;
    // (the empty statement keeps these loads ahead of the branch; the values every lane holds alike go back to scalars)
    asm volatile("" : "+v"(M), "+v"(K), "+v"(area), "+v"(sym_rep), "+v"(sym_rep_hi), "+v"(sym_len), "+v"(sym_code));
    M = __builtin_amdgcn_readfirstlane(M); K = __builtin_amdgcn_readfirstlane(K);
    area = ((u64)__builtin_amdgcn_readfirstlane((u32)(area >> 32)) << 32) | __builtin_amdgcn_readfirstlane((u32)area);
    if ((verdict >> 8) == epoch || first >= nchunks) return;
    // the offset-table entries of this wavefront's next 64 chunks, one chunk per lane
    const u32* off_tab = reinterpret_cast<const u32*>(blob + kHeaderBytes);
    u32 off0 = 0, off1 = 0;
    auto fetch_offsets = [&](u64 from) {
        const u64 c = from + (u64)lane * stride;
        if (c < nchunks) { off0 = off_tab[c]; off1 = off_tab[c + 1]; }
    };
    fetch_offsets(first);
    uint4* pay = dec_pay + wave * (pay_words / 4 + 1);
    u32* ring = VERIFY ? s_ring : s_ring + wave * kRingWords * kW;
    const u32 zero_bits = zero_chunk_bits(read_lane(sym_len, K), read_lane(sym_code, K));
    auto raise = [&](u32 code) { raise_status(ws, host, epoch, code); };
    // A wavefront brings the tables to LDS when it comes to the first chunk that has to be decoded (in a sparse blob most
    // never do).  Each does so for itself: they all write the same values to the same places, and none waits for another.
    bool have_tables = false;
    CodeLens lens;
    QuietChunk q;
    u32 turn = 0, c = first, o0 = read_lane(off0, 0), o1 = read_lane(off1, 0);
    q.start(blob, area, o0, o1, zero_bits, (u64)(c + 1) * kChunk <= n);
    while (true) {
        const bool full = (u64)(c + 1) * kChunk <= n;
        const bool quiet = q.holds(zero_bits);
        const u64 cn = (u64)c + stride;
        const bool more = cn < nchunks;
        u32 n0 = 0, n1 = 0;
        if (more) {
            ++turn;
            if ((turn & (kW - 1)) == 0) fetch_offsets(cn);
            n0 = read_lane(off0, turn & (kW - 1)); n1 = read_lane(off1, turn & (kW - 1));
            q.start(blob, area, n0, n1, zero_bits, (cn + 1) * kChunk <= n);
        }
        if (!quiet) {
            if (!have_tables) {
                have_tables = true;
                u32x4 e[(1u << kMultiBits) / 4 / kW];
#pragma unroll
                for (u32 k = 0; k < (1u << kMultiBits) / 4 / kW; ++k) e[k] = reinterpret_cast<const u32x4*>(D.multi)[lane + k * kW];
#pragma unroll
                for (u32 k = 0; k < (1u << kMultiBits) / 4 / kW; ++k) reinterpret_cast<u32x4*>(L.multi)[lane + k * kW] = e[k];
                if (lane < kMaxSym) {
                    L.rep[lane] = __uint_as_float(lane < K ? sym_rep : 0x80000000u);
                    L.rep64[lane] = lane < K ? __hiloint2double((int)sym_rep_hi, (int)sym_rep) : -0.0;
                }
                if (M > kMultiBits) build_longs(L, sym_len, sym_code);
                lens.set(sym_len, K);
                __builtin_amdgcn_wave_barrier();
            }
            decode_chunk<DT, VERIFY>(blob, w_ref, n, c, o0, o1, full, M > kMultiBits, ahead != 0, L, pay, pay_words, ring, K, lens, area, raise);
        }
        if (!more) break;
        c = (u32)cn; o0 = n0; o1 = n1;
    }
}

// ----------------------------------------------------------------------------- batched decode
// lc_decode_batch: the blobs of many tensors restored in three launches (five and a copy before: 161 tensors 90 -> 83 us).  Every blob is validated as
// lc_decode validates it (header and symbol table per tensor, then every chunk's place in its offset
// table) before the sweep; a tensor whose blob fails is left untouched and reported, the others are
// restored.  The sweep deals the chunks of all tensors round-robin to single-wavefront workgroups,
// which reload their look-up tables when they move on to another tensor's chunk.
// One workgroup per tensor: what the host says about it (read from mapped host memory, kept for the kernels behind this one: a
// copy of the list to the device ahead of the call took longer than that read), which chunks are its own, header, symbol
// table, codes, look-up table, and its outcome so far, for the host as well.
__global__ __launch_bounds__(256) void kb_dec_tables(BatchDecArgs a) {
    __shared__ u32 hdr[kHeaderBytes / 4];
    __shared__ u32 s_ok;
    __shared__ DecBuild B;
    const u32 t = threadIdx.x, sidx = blockIdx.x;
    __shared__ SegD sg;
    if (t < sizeof(SegD) / 4) reinterpret_cast<u32*>(&sg)[t] = reinterpret_cast<const u32*>(a.host_segs + sidx)[t];
    __syncthreads();
    if (t < sizeof(SegD) / 4) reinterpret_cast<u32*>(a.segs + sidx)[t] = reinterpret_cast<const u32*>(&sg)[t];
    for (u32 c = t; c < sg.nchunks; c += 256) a.seg_of_chunk[sg.chunk0 + c] = sidx;
    DecSet& D = a.sets[sidx];
    if (t < kHeaderBytes / 4) hdr[t] = reinterpret_cast<const u32*>(sg.blob)[t];
    __syncthreads();
    if (t < kW) {
        const u64 hn = hdr[2] | ((u64)hdr[3] << 32), total = hdr[10] | ((u64)hdr[11] << 32);
        const u64 area = chunk_area_of(sg.nchunks);
        // the largest blob lc_encode can produce for this n (nbits 4): header + offsets + 132 bytes per chunk + n/2
        const u64 max_total = area + (u64)sg.nchunks * (2 * kW + 4) + (sg.n * 4 + 7) / 8;
        const bool sound = hdr[0] == 0x3142434Cu && hdr[1] == (1u | (kHeaderBytes << 16)) && hdr[12] == 0;
        const bool head_ok = sound && hn == sg.n && hdr[15] == (u32)a.dtype && hdr[9] == sg.nchunks && total >= area &&
                             total <= max_total && ((total - area) & 3) == 0;
        bool ok = head_ok;
        u32 status = 0;
        if (!head_ok) status = (sound && (hn != sg.n || hdr[15] != (u32)a.dtype)) ? 1u : 4u;
        else if (!dec_symbol_table(hdr, sg.n, sg.nchunks, area, (total - area) / 4, D, B)) { ok = false; status = 4u; }
        if (t == 0) {
            if (!ok) { D.info.area = 0; D.info.total_words = 0; D.info.max_len = 0; D.info.K = 0; }
            a.seg_status[sidx] = status;
            a.results[sidx].bytes = ok ? total : 0; a.results[sidx].status = status; a.results[sidx].used_cache = 0;
            D.info.pad[0] = ok ? 1u : 0u;                    // the chunk checks and the sweep look here first
            D.info.pad[1] = 0;
            s_ok = ok;
        }
    }
    __syncthreads();
    if (s_ok) dec_build_luts(D, B, hdr[5], t);
}

// A finding in a tensor's chunks: gates its sweep, and tells the host (any finding will do).
__device__ __forceinline__ void batch_raise(const BatchDecArgs& a, u32 sidx, u32 status) {
    atomicMax(&a.seg_status[sidx], status);
    a.results[sidx].status = status;
}

// Also leaves, per chunk, what the sweep needs to find it: {tensor, chunk index there, the chunk's two offset-table
// entries}, so that the sweep's wavefronts get each chunk's place with one load that they can issue a chunk ahead.
__global__ __launch_bounds__(256) void kb_dec_chunks(BatchDecArgs a) {
    const u32 g = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (g >= a.total_chunks) return;
    const u32 sidx = a.seg_of_chunk[g];
    const SegD& sg = a.segs[sidx];
    const DecInfo& I = a.sets[sidx].info;
    const u32 c = g - sg.chunk0;
    uint4 info = make_uint4(sidx, c, 0u, 0u);
    if (I.pad[0]) {                                   // (a blob whose header failed: its tensor's status says so, the sweep skips it)
        const u32* off_tab = reinterpret_cast<const u32*>(sg.blob + kHeaderBytes);
        info.z = off_tab[c]; info.w = off_tab[c + 1];
        if (!dec_chunk_ok(sg.blob, I.area, I.total_words, sg.nchunks, c) && lane_id() == 0) batch_raise(a, sidx, 4u);
    }
    if (lane_id() == 0) reinterpret_cast<uint4*>(a.chunk_info)[g] = info;
}

template <int DT>
__global__ __launch_bounds__(64) void kb_decode(BatchDecArgs a) {
    __shared__ DecLds L;
    __shared__ u32 ring[kRingWords * kW];
    __shared__ uint4 pay[kPayWords / 4 + 1];
    const u32 lane = threadIdx.x;
    u32 active = 0xFFFFFFFFu, M = 0, K = 0, zero_bits = 0;
    bool have_tables = false;
    CodeLens lens;
    u64 area = 0;
    const uint4* chunk_info = reinterpret_cast<const uint4*>(a.chunk_info);
    auto info_of = [&](u32 g) {                      // (the same in every lane: back to scalar registers)
        uint4 q = g < a.total_chunks ? chunk_info[g] : make_uint4(0u, 0u, 0u, 0u);
        q.x = __builtin_amdgcn_readfirstlane(q.x); q.y = __builtin_amdgcn_readfirstlane(q.y);
        q.z = __builtin_amdgcn_readfirstlane(q.z); q.w = __builtin_amdgcn_readfirstlane(q.w);
        return q;
    };
    uint4 next = info_of(blockIdx.x);
    for (u32 g = blockIdx.x; g < a.total_chunks; g += gridDim.x) {
        const uint4 info = next;
        next = info_of(g + gridDim.x);               // on its way while this chunk is decoded
        const u32 sidx = info.x;
        // a tensor whose blob failed a check is not touched
        if (__hip_atomic_load(&a.seg_status[sidx], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) continue;
        const SegD& sg = a.segs[sidx];
        const DecSet& D = a.sets[sidx];
        if (sidx != active) {
            active = sidx;
            have_tables = false;
            M = D.info.max_len; K = D.info.K; area = D.info.area;
            zero_bits = zero_chunk_bits(D.info.len[K], D.info.code[K]);
        }
        auto raise = [&](u32 code) { batch_raise(a, sidx, code); };
        const u32 c = info.y, o0 = info.z, o1 = info.w;
        const bool full = (u64)(c + 1) * kChunk <= sg.n;
        QuietChunk q;
        q.start(sg.blob, area, o0, o1, zero_bits, full);
        if (q.holds(zero_bits)) continue;
        if (!have_tables) {
            // (brought to LDS for the first chunk of the tensor that has to be decoded)
            have_tables = true;
            u32x4 e[(1u << kMultiBits) / 4 / kW];
            u32 rep = 0, len = 0, code = 0;
#pragma unroll
            for (u32 k = 0; k < (1u << kMultiBits) / 4 / kW; ++k) e[k] = reinterpret_cast<const u32x4*>(D.multi)[lane + k * kW];
            if (lane < kMaxSym) { rep = D.info.rep_bits[lane]; len = D.info.len[lane]; code = D.info.code[lane]; }
#pragma unroll
            for (u32 k = 0; k < (1u << kMultiBits) / 4 / kW; ++k) reinterpret_cast<u32x4*>(L.multi)[lane + k * kW] = e[k];
            if (lane < kMaxSym) { L.rep[lane] = __uint_as_float(lane < K ? rep : 0x80000000u); }
            if (M > kMultiBits) build_longs(L, len, code);
            lens.set(len, K);
            __builtin_amdgcn_wave_barrier();
        }
        decode_chunk<DT>(sg.blob, sg.w_ref, sg.n, c, o0, o1, full, M > kMultiBits, true, L, pay, kPayWords, ring, K, lens, area, raise);
    }
}

// ----------------------------------------------------------------------------- k_decode_fused
// Restore from several checkpoints in one sweep (Section 3, C1: u_t = u_0 + sum of the decoded
// deltas; Section 3.2, checkpoint merging): up to kMaxMany blobs of the same n are decoded side
// by side and their values added to w_ref in blob order, one fp32 add per blob and element, so
// the result equals that of applying the blobs one call after the other, with one read and
// one write of w_ref instead of one per blob.
// T is a compile-time constant, so the T bit strings of a
// lane are T independent dependency chains that the scheduler interleaves.  One wavefront per
// workgroup; the payloads of a chunk (all T blobs) are staged in the workgroup's LDS area with
// coalesced loads (the host sizes the area to the blobs, which also sets how many wavefronts
// share a compute unit).  With codes of at most 7 bits (always the case for nbits <= 3) a row's 4 codes
// of one blob take at most 28 bits, so each blob's 32-bit window is re-read once per row from the bit
// position alone, without a branch; with longer codes (LONG) twice per row.  Both look-up
// tables are free of LDS bank conflicts: 128 one-byte entries over the next 7 bits (code length
// and symbol), then the symbol's representative.  A chunk whose payloads do not fit the LDS
// area reads them from memory instead.
template <int T>
struct FusedHead {
    uint16_t lut[T][1u << kDecLut1Bits];         // next 7 bits -> e = (len << 4 | symbol) << 2
    u32 rep[T][128];                             // byte offset e -> representative bits (-0.0: merged symbol); a symbol
                                                 // has one length, so distinct entries in use lie in distinct banks
    const uint8_t* rec_base[T];                  // start of the chunk records
    const u32* off_tab[T];
    // Codes longer than the 7 bits of lut (its entry is then kFusedEscape): the symbols in canonical order
    // (shorter codes first, then by index) have increasing left-justified codes, so the rank of the symbol a
    // window starts with is the number of codes not above the window; only the long ones need comparing.
    u32 lj[T][kMaxSym];                          // rank -> code, left-justified in 32 bits
    uint16_t e_rank[T][kMaxSym];                 // rank -> (len << 4 | symbol) << 2
    u32 rep_sym[T][kMaxSym];                     // symbol -> representative bits
    u32 first_long[(T + 3) / 4 * 4];             // rank of the first code longer than 7 bits
    u32 nranks[(T + 3) / 4 * 4];                 // symbols with a code
    u32 zero_bits[(T + 3) / 4 * 4];              // per blob: lane length of a chunk of merged symbols only (0: never skip)
    u32 pad[3];
    u32 before_pay;                              // the word in front of the payload area (read, never used)
};
constexpr u32 kFusedEscape = 0xFFu << 2;         // what lut holds for a prefix of a longer code (no short entry has length 15)
constexpr u32 kFusedSlack = 128;                 // words behind the payloads that a damaged lane string may run into:
                                                 // 256 codes of at most 15 bits past a start that validation bounds

// Bit positions are kept as p = 31 + bits from the start of the payload area (staged) or of the
// blob's payload (from memory): the window is then the low 32 bits of {word[(p >> 5) - 1],
// word[p >> 5]} >> (~p & 31), which is one v_alignbit.
// LONG: some blob of the sweep has codes longer than 7 bits.  Two codes then take up to 30 bits, so the window is
// re-read after the second code of a row, and a window that starts with a long code is ranked against the long
// codes (a handful of compares; rare, since long codes belong to rare symbols).
template <int T, bool FAST, bool STAGED, bool LONG, int DT>
__device__ __forceinline__ void fused_row(const FusedHead<T>& H, const u32* pay, u32 pay_words, const u32* const (&gw)[T],
                                          const u32 (&nw)[T], u32 (&pos)[T], void* __restrict__ w_ref, u64 n, u64 idx,
                                          float (&x)[4]) {
    // Written step by step across the blobs (all windows, then the first code of every blob, ...), so
    // that the T look-ups of a step are in flight together.
    u32 win[T], rep[4][T];
    auto windows = [&]() {
#pragma unroll
        for (int t = 0; t < T; ++t) {
            u32 hi, lo;                                   // the two payload words around the lane's position
            if (STAGED) {
                const u32 wi = pos[t] >> 5;              // stays inside the area and its slack
                hi = pay[(int)wi - 1]; lo = pay[wi];
            } else {
                const u32 wi = pos[t] >> 5, last = nw[t] - 1;
                hi = wi ? gw[t][min(wi - 1, last)] : 0u; lo = gw[t][min(wi, last)];
            }
            win[t] = __builtin_amdgcn_alignbit(hi, lo, ~pos[t]);
        }
    };
    windows();
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        if (LONG && v == 2) windows();
        if (FAST || idx + v < n) {
            u32 e[T];
#pragma unroll
            for (int t = 0; t < T; ++t) {
                e[t] = H.lut[t][win[t] >> (32 - kDecLut1Bits)];
                asm("" : "+v"(e[t]));                 // keep e a 32-bit value (no 16-bit shift plus re-extension)
            }
            if (LONG) {
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    if (__any(e[t] == kFusedEscape)) {
                        const u32 first = H.first_long[t], nr = H.nranks[t];
                        u32 r = first;
                        for (u32 j = first + 1; j < nr; ++j) r += win[t] >= H.lj[t][j] ? 1u : 0u;
                        if (e[t] == kFusedEscape) e[t] = H.e_rank[t][r];
                    }
                }
            }
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const u32 len = e[t] >> 6;
                if (LONG) rep[v][t] = H.rep_sym[t][(e[t] >> 2) & 15u];
                else rep[v][t] = *reinterpret_cast<const u32*>(reinterpret_cast<const uint8_t*>(H.rep[t]) + e[t]);
                win[t] <<= len; pos[t] += len;
            }
        } else {
#pragma unroll
            for (int t = 0; t < T; ++t) rep[v][t] = 0x80000000u;
        }
    }
    u32 kept = 1;                                     // a single blob often leaves whole rows unchanged: skip their write
    if (T == 1) kept = (rep[0][0] | rep[1][0] | rep[2][0] | rep[3][0]) & 0x7FFFFFFFu;
    if (FAST) {
        if (T > 1 || __any(kept != 0)) {
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int t = 0; t < T; ++t) x[v] = stored<DT>(__fadd_rn(x[v], __uint_as_float(rep[v][t])));   // in blob order
            // (binary32 rows as a plain float4 store: with non-temporal stores, or with the same 16 bytes stored through
            // a compiler vector type, the first sweep over parameters that a device copy had just written took 830-880 us
            // instead of 600-650)
            if constexpr (DT == kF32) *reinterpret_cast<float4*>(static_cast<float*>(w_ref) + idx) = make_float4(x[0], x[1], x[2], x[3]);
            else store4<DT>(w_ref, idx, x);
        }
    } else {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            if (idx + v < n) {
#pragma unroll
                for (int t = 0; t < T; ++t) x[v] = stored<DT>(__fadd_rn(x[v], __uint_as_float(rep[v][t])));
                store_one<DT>(w_ref, idx + v, x[v]);
            }
        }
    }
}

// All rows of a chunk with staged payloads: w_ref is read PF rows ahead in two
// alternating register batches, so the reads of the next rows are in flight while these decode.  Of a ragged chunk (not FULL),
// which is one wavefront's work from start to end and the sweep's last, the whole rows go the same way, only what is left of it
// element by element: by elements from the first row on, with payloads from memory, fp32, a blob of 738 chunks less 777 elements took
// 77 us the call, and 61 so, 8 blobs of 1 to 15 chunks 139 and 97, 12 of 1,197 chunks 397 and 262.
template <int T, bool FULL, bool LONG, int DT>
__device__ __forceinline__ void fused_rows_fast(const FusedHead<T>& H, const u32* pay, u32 pay_words, const u32* const (&gw)[T],
                                                const u32 (&nw)[T], u32 (&pos)[T], void* __restrict__ w_ref, u64 n, u32 c) {
    constexpr int PF = 4;
    typedef typename Raw<DT>::type RowT;
    const u32 lane = lane_id();
    const u64 base = (u64)c * kChunk + lane * kV;
    const u32 rows = FULL ? kR : (u32)(n - (u64)c * kChunk) / kRowElems;
    RowT A[PF], B[PF];
    auto fetch = [&](RowT (&X)[PF], u32 r0) {
#pragma unroll
        for (int k = 0; k < PF; ++k)                      // (no branch, or the loads would be waited for: the last whole row again)
            X[k] = load_raw<DT>(w_ref, base + (u64)(FULL ? r0 + k : min(r0 + k, rows - 1)) * kRowElems);
    };
    auto batch = [&](RowT (&X)[PF], u32 r0) {
#pragma unroll
        for (int k = 0; k < PF; ++k) {
            if (!FULL && r0 + k >= rows) break;
            float x[4];
            unpack<DT>(X[k], x);
            fused_row<T, true, true, LONG, DT>(H, pay, pay_words, gw, nw, pos, w_ref, n, base + (u64)(r0 + k) * kRowElems, x);
        }
    };
    if (FULL || rows > 0) fetch(A, 0);
    for (u32 r0 = 0; r0 < rows; r0 += 2 * PF) {
        fetch(B, r0 + PF);
        batch(A, r0);
        if (r0 + 2 * PF < kR) fetch(A, r0 + 2 * PF);
        batch(B, r0 + PF);
    }
    if (!FULL) {
        const u64 idx = base + (u64)rows * kRowElems;
        float x[4];
        load_row<false, DT>(w_ref, idx, n, x);
        fused_row<T, false, true, LONG, DT>(H, pay, pay_words, gw, nw, pos, w_ref, n, idx, x);
    }
}

// A chunk whose payloads are read from memory, row by row.
template <int T, bool FAST, bool LONG, int DT>
__device__ __forceinline__ void fused_rows_plain(const FusedHead<T>& H, const u32* const (&gw)[T], const u32 (&nw)[T], u32 (&pos)[T],
                                              void* __restrict__ w_ref, u64 n, u32 c) {
    const u32 lane = lane_id();
    const u64 base = (u64)c * kChunk;
    for (u32 r = 0; r < kR; ++r) {
        const u64 idx = base + (u64)r * kRowElems + lane * kV;
        if (!FAST && idx >= n) break;
        float x[4];
        load_row<FAST, DT>(w_ref, idx, n, x);
        fused_row<T, FAST, false, LONG, DT>(H, nullptr, 0, gw, nw, pos, w_ref, n, idx, x);
    }
}

template <typename P>
__device__ __forceinline__ P* uniform_ptr(P* p) {        // a pointer every lane holds alike, moved to scalar registers
    const u64 v = reinterpret_cast<u64>(p);
    const u32 lo = __builtin_amdgcn_readfirstlane((u32)v), hi = __builtin_amdgcn_readfirstlane((u32)(v >> 32));
    return reinterpret_cast<P*>(((u64)hi << 32) | lo);
}

template <int T, bool LONG, int DT>
__device__ __forceinline__ void fused_chunk(const FusedHead<T>& H, u32* pay, u32 pay_words, void* __restrict__ w_ref, u64 n,
                                            Workspace* ws, HostResult* host, u32 c, u32 nchunks, u64 epoch) {
    const u32 lane = lane_id();
    const bool full = (u64)(c + 1) * kChunk <= n;
    const u32* gw[T];
    u32 nw[T], k0[T], wbase[T], pos[T], start[T], lane_bits[T];
    u32 total = 0;
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const u32* ot = uniform_ptr(H.off_tab[t]);
        const u32 o0 = ot[c], o1 = ot[c + 1];
        const uint8_t* rec = uniform_ptr(H.rec_base[t]) + 4 * (u64)o0;
        nw[t] = o1 - o0 - kLaneBitsWords;                 // >= 1 (validated)
        lane_bits[t] = reinterpret_cast<const uint16_t*>(rec)[lane];
        gw[t] = reinterpret_cast<const u32*>(rec + 2 * kW);
        k0[t] = (u32)((reinterpret_cast<uintptr_t>(gw[t]) >> 2) & 3);
        wbase[t] = total;
        total += (nw[t] + k0[t] + 3) & ~3u;
    }
    const bool staged = total <= pay_words;
    if (staged) {
        // Coalesced copies of [16-byte aligned start, payload end) into the LDS area; the words before a
        // payload are its record's lane lengths.  A last partial vector may read up to 12 bytes past the
        // payload: into the next record, except in the last chunk, which reads that vector word by word.
        constexpr int CV = T > 4 ? 2 : 4;                 // vectors per lane and blob in flight
        const bool guard = c + 1 == nchunks;
        u32 most = 0;
#pragma unroll
        for (int t = 0; t < T; ++t) most = max(most, (nw[t] + k0[t] + 3) >> 2);
        u32 nonzero = 0;                                  // OR of this lane's share of the payload words
        for (u32 i0 = 0; i0 < most; i0 += CV * kW) {
            uint4 q[T][CV];
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const uint4* gv = reinterpret_cast<const uint4*>(gw[t] - k0[t]);
                const u32 have = nw[t] + k0[t], nvec = (have + 3) >> 2;
#pragma unroll
                for (int k = 0; k < CV; ++k) {
                    const u32 i = i0 + k * kW + lane;
                    if (i < nvec) {
                        if (!guard || 4 * i + 4 <= have) q[t][k] = gv[i];
                        else {
                            const u32* tw = reinterpret_cast<const u32*>(gv + i);
                            const u32 left = have - 4 * i;
                            q[t][k].x = tw[0]; q[t][k].y = left > 1 ? tw[1] : 0; q[t][k].z = left > 2 ? tw[2] : 0; q[t][k].w = 0;
                        }
                    }
                }
            }
#pragma unroll
            for (int t = 0; t < T; ++t) {
                uint4* dst = reinterpret_cast<uint4*>(pay + wbase[t]);
                const u32 have = nw[t] + k0[t], nvec = (have + 3) >> 2;
#pragma unroll
                for (int k = 0; k < CV; ++k) {
                    const u32 i = i0 + k * kW + lane;
                    if (i < nvec) {
                        dst[i] = q[t][k];
                        const u32 j = 4 * i;              // words [k0, have) of the copied range are payload
                        nonzero |= (j >= k0[t] && j < have ? q[t][k].x : 0u) | (j + 1 >= k0[t] && j + 1 < have ? q[t][k].y : 0u) |
                                   (j + 2 >= k0[t] && j + 2 < have ? q[t][k].z : 0u) | (j + 3 >= k0[t] && j + 3 < have ? q[t][k].w : 0u);
                    }
                }
            }
        }
        // every blob's chunk holds merged symbols only (see zero_chunk_bits; a ragged chunk's lanes are not alike): nothing changes,
        // w_ref is not read
        bool all_merged = full;
#pragma unroll
        for (int t = 0; t < T; ++t) all_merged = all_merged && H.zero_bits[t] != 0 && lane_bits[t] == H.zero_bits[t];
        if (!__any(!all_merged || nonzero != 0)) return;
    }
#pragma unroll
    for (int t = 0; t < T; ++t) start[t] = 31 + wave_incl_scan(lane_bits[t]) - lane_bits[t];
    if (staged) {
#pragma unroll
        for (int t = 0; t < T; ++t) { start[t] += 32 * (wbase[t] + k0[t]); pos[t] = start[t]; }
        if (full) fused_rows_fast<T, true, LONG, DT>(H, pay, pay_words, gw, nw, pos, w_ref, n, c);
        else fused_rows_fast<T, false, LONG, DT>(H, pay, pay_words, gw, nw, pos, w_ref, n, c);
    } else {
#pragma unroll
        for (int t = 0; t < T; ++t) pos[t] = start[t];
        if (full) fused_rows_plain<T, true, LONG, DT>(H, gw, nw, pos, w_ref, n, c);
        else fused_rows_plain<T, false, LONG, DT>(H, gw, nw, pos, w_ref, n, c);
    }
    bool bad = false;
#pragma unroll
    for (int t = 0; t < T; ++t) bad = bad || (pos[t] - start[t] != lane_bits[t]);
    if (__any(bad) && lane == 0) raise_status(ws, host, epoch, 4u);
}

// Wavefronts per SIMD that the registers leave, where the LDS does too, with sparse blobs (4 of them, two of 1 % kept symbols, one
// unchanged, fp32, 5,919 chunks with one wavefront per SIMD less 235 us and 195, 2^27 elements 318 and 263), and may leave: of 4 dense
// blobs 8 wavefronts fit a compute unit, which with 2-byte elements had better be 2 per SIMD than 3 on some (1,831 chunks that no cache
// holds 95 us and 104).
constexpr bool fused_twos(int blobs, bool long_codes, int dt) { return blobs == 4 && !long_codes && dt != kF32; }
constexpr int fused_waves(int blobs, bool long_codes, int dt) {
    return blobs <= 2 || (blobs == 3 && long_codes && dt == kF32) ? 4 : blobs <= 5 && !fused_twos(blobs, long_codes, dt) ? 3 : 2;
}
template <int T, bool LONG, int DT>
__global__ __launch_bounds__(64) LC_WAVES_PER_SIMD(fused_waves(T, LONG, DT), fused_twos(T, LONG, DT) ? 2 : 8)
void k_decode_fused(BlobList blobs, u32 first, void* __restrict__ w_ref, u64 n, Workspace* ws, u32 nchunks, u64 epoch, HostResult* host,
                    u32 pay_words) {
    __shared__ FusedHead<T> H;
    static_assert(sizeof(FusedHead<T>) % 16 == 0, "payload area must stay 16-byte aligned");
    extern __shared__ uint4 fused_pay[];                 // pay_words + kFusedSlack payload words, right behind H
    u32* pay = reinterpret_cast<u32*>(fused_pay);
    // if a check found something, touch nothing
    if ((__hip_atomic_load(&ws->dec_status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> 8) == epoch) return;
    const u32 tid = threadIdx.x;
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const DecSet& D = ws->dec_set[first + t];
        const u32 M = D.info.max_len, K = D.info.K;       // entries of codes of at most 7 bits: e < 512
        const u32 P1 = M < kDecLut1Bits ? M : kDecLut1Bits;
        for (u32 i = tid; i < (1u << kDecLut1Bits); i += kW) {
            const u32 e = D.lut1[i >> (kDecLut1Bits - P1)];
            H.lut[t][i] = (uint16_t)(e << 2);
            H.rep[t][i] = (i & 15) < K ? D.info.rep_bits[i & 15] : 0x80000000u;
        }
        if (LONG && tid < kMaxSym) {
            // this symbol's rank in canonical order (shorter codes first, then by index)
            const u32 j = tid, own = D.info.len[j];
            u32 rank = 0, coded = 0, short_codes = 0;
            for (u32 i = 0; i < kMaxSym; ++i) {
                const u32 li = D.info.len[i];
                if (li == 0) continue;
                ++coded;
                if (li <= kDecLut1Bits) ++short_codes;
                if (own && (li < own || (li == own && i < j))) ++rank;
            }
            H.rep_sym[t][j] = j < K ? D.info.rep_bits[j] : 0x80000000u;
            if (own) { H.lj[t][rank] = D.info.code[j] << (32 - own); H.e_rank[t][rank] = (uint16_t)(((own << 4) | j) << 2); }
            if (tid == 0) { H.first_long[t] = short_codes; H.nranks[t] = coded; }
        }
        if (tid == 0) {
            const uint8_t* blob = blobs.p[first + t];
            H.zero_bits[t] = zero_chunk_bits(D.info.len[K], D.info.code[K]);
            H.rec_base[t] = blob + D.info.area;
            H.off_tab[t] = reinterpret_cast<const u32*>(blob + kHeaderBytes);
        }
    }
    if (tid == 0) H.before_pay = 0;
    __syncthreads();
    for (u32 c = blockIdx.x; c < nchunks; c += gridDim.x) fused_chunk<T, LONG, DT>(H, pay, pay_words, w_ref, n, ws, host, c, nchunks, epoch);
}
// ----------------------------------------------------------------------------- k_decode_pairs
// The same for more blobs in one sweep, up to 8 where the other kernel takes 4 (dense ones; of sparse ones some 6).  What stands in the way of
// that is the LDS: with the payloads of whole chunks in it, 8 blobs leave room for 4 wavefronts, one per SIMD, each of which waits out its own
// look-ups (8 blobs of 355 M elements 1,470 us, two sweeps of 4 by the other kernel 1,240).
// - Of its strings a lane has a window of kWords words per blob in LDS, 2 KB per blob and wavefront: two wavefronts per SIMD.  A
//   lane's windows lie in a bank of its own, so that no two lanes meet when they read at places of their own; a read at any
//   place of a whole payload costs the LDS 7 cycles instead of 2.6.
// - The windows move on a few at a time, the words asked for 4 rows ahead and ahead of the rows of w_ref (a wait for them, in
//   order, would else wait for those rows as well: 1,140 us, 930 so); a blob whose windows some lane would leave within two rows
//   is served at once.  A string is read some four times that way, all of it past the L2: 2 GB beside 3.4.
// - A step takes two symbols: one look-up over the next 10 bits gives both and their length together, one more their two
//   representatives (8 bytes at an aligned place cost the LDS hardly more than 4).  18 vector and 5 LDS instructions per row of
//   4 symbols and blob; one symbol per look-up took 24 and 9.
// 8 blobs of 355 M elements, codes of 1.65 bits: 1,240 us in two sweeps, 930 so; vector issue 51 %, LDS 56 % of its cycles, and
// 5.6 TB/s past the L2.  Without the windows' words it would take 740, without w_ref 750.
// WIDE: some blob of the sweep has more than 8 symbols: pairs of 4-bit symbols, 11 bits to look up, since its codes
// are longer, and twice the words.  Two codes that do not fit the table's bits (under 0.1 % of the pairs of codes of
// 1.7 bits on average, 0.3 % of those of 3.5; most of them in a layer whose symbols are all rare ones) are told from their
// entry and taken one by one.
// Arrays that are off alignment take the same loads and stores.
constexpr u32 kPairsWaves = 8;
constexpr u32 kPairEscape = 0x8000;
template <int T, bool WIDE>
struct PairsLds {
    static constexpr u32 kBits = WIDE ? 11 : 10, kSym = WIDE ? 4 : 3, kSyms = 1u << kSym;
    static constexpr u32 kWords = WIDE ? 16 : 8;
    static constexpr u32 kTurns = T > 4 ? 4 : 2;                           // windows that may move on at a time
    static constexpr u32 kStepBits = 2 * kV * (WIDE ? 15 : 7);             // the most that two rows take
    lc_f32x2 rep[T][kSyms * kSyms];                // first symbol | second << kSym -> representatives (-0.0: merged symbol)
    alignas(16) uint16_t lut[T][1u << kBits];    // next bits -> that index | length of both << 8; or kPairEscape | first symbol |
                                                 // its length << 8 (0: longer than the table's bits)
    // Codes one by one: the symbols in canonical order (shorter codes first, then by index) have increasing left-justified
    // codes, so the rank of the symbol a window starts with is the number of codes not above the window.
    alignas(16) u32 lj[T][kSyms];                // rank -> code, left-justified in 32 bits
    u32 e_rank[T][kSyms];                        // rank -> len << 4 | symbol
    u32 len[T][kSyms];                           // of every symbol
    const uint8_t* rec_base[T];                  // start of the chunk records
    const u32* off_tab[T];
    u32 nranks[T], merged[T];                    // symbols with a code; the merged symbol
    u32 zero_bits[T];                            // lane length of a chunk of merged symbols only (0: never skip)
    u32 stop, taken;                             // chunks that its wavefronts have taken
    // word k of lane l's window of blob t: [wave][t][k][l] (the word in front of a window is read, never used)
    alignas(kWords * 256) u32 win[kPairsWaves][T][kWords][kW];
};

// A wavefront's places in one chunk's strings.  p: 31 + bits from the start of a window's words, which start at word `from`
// of the blob's payload of this chunk.
template <int T, bool WIDE>
struct PairsStrings {
    typedef PairsLds<T, WIDE> Lds;
    const u32* gw[T];                            // the payloads in memory
    u32 nw[T];                                   // and their words
    u32 p[T], from[T];
    // The window's next 32 bits: the low half of {word[(p >> 5) - 1], word[p >> 5]} >> (~p & 31).  (A damaged string may run on;
    // its words are then any of the window's.)
    static __device__ __forceinline__ u32 next(const Lds& L, u32 wave, int t, u32 p) {
        const u32 at = ((p << 3) & ((Lds::kWords - 1) * 256)) | (lane_id() * 4);
        const u32* w = reinterpret_cast<const u32*>(reinterpret_cast<const uint8_t*>(&L.win[wave][t][0][0]) + at);
        return __builtin_amdgcn_alignbit(*(w - kW), *w, ~p);
    }
};

// A window's words on their way.
template <int T, bool WIDE>
struct PairsWords {
    static constexpr u32 kVecs = PairsLds<T, WIDE>::kWords / 4;
    typedef u32x4 __attribute__((aligned(4))) vec_any;
    u32x4 q[kVecs];
    u32 from;
    // A window may reach past the payload into the next record, which is longer; in the blob's last chunk (last) it may not.
    __device__ __forceinline__ void fetch(const PairsStrings<T, WIDE>& S, int t, bool last) {
        from = min(S.from[t] + ((S.p[t] - 31) >> 5), S.nw[t]);
        if (!last) {
            const u32* w = S.gw[t] + from;
#pragma unroll
            for (u32 k = 0; k < kVecs; ++k) q[k] = *reinterpret_cast<const vec_any*>(w + 4 * k);
        } else {
            const u32 end = S.nw[t] - 1;
#pragma unroll
            for (u32 k = 0; k < kVecs; ++k) {
                const u32 f = from + 4 * k;
                q[k] = u32x4{S.gw[t][min(f, end)], S.gw[t][min(f + 1, end)], S.gw[t][min(f + 2, end)], S.gw[t][min(f + 3, end)]};
            }
        }
    }
    __device__ __forceinline__ void place(PairsStrings<T, WIDE>& S, PairsLds<T, WIDE>& L, u32 wave, int t) const {
        u32* w = &L.win[wave][t][0][lane_id()];
#pragma unroll
        for (u32 k = 0; k < kVecs; ++k) { w[(4 * k) * kW] = q[k].x; w[(4 * k + 1) * kW] = q[k].y; w[(4 * k + 2) * kW] = q[k].z; w[(4 * k + 3) * kW] = q[k].w; }
        S.p[t] += 32 * (S.from[t] - from);
        S.from[t] = from;
    }
};

// The symbol a window starts with: len << 4 | symbol (a prefix that starts no code: the merged symbol, length 0).
template <int T, bool WIDE>
__device__ __forceinline__ u32 pairs_one(const PairsLds<T, WIDE>& L, int t, u32 win) {
    u32 r = 0;
    u32x4 lj[PairsLds<T, WIDE>::kSyms / 4];                  // (all of them asked for at once: behind the last code, all ones)
#pragma unroll
    for (u32 k = 0; k < PairsLds<T, WIDE>::kSyms / 4; ++k) lj[k] = reinterpret_cast<const u32x4*>(L.lj[t])[k];
#pragma unroll
    for (u32 k = 0; k < PairsLds<T, WIDE>::kSyms / 4; ++k) r += (win >= lj[k].x) + (win >= lj[k].y) + (win >= lj[k].z) + (win >= lj[k].w);
    r = min(r, L.nranks[t]) - 1;                             // (the first code is 0)
    const u32 e = L.e_rank[t][r];
    return ((win ^ L.lj[t][r]) >> (32 - (e >> 4))) == 0 ? e : L.merged[t];
}

// Two symbols that do not fit the table together, as an entry of it (of up to 30 bits); e: what it holds for the window's bits.
template <int T, bool WIDE>
__device__ __forceinline__ u32 pairs_slow(const PairsLds<T, WIDE>& L, u32 wave, int t, u32 p, u32 win, u32 e) {
    constexpr u32 kBits = PairsLds<T, WIDE>::kBits, kSym = PairsLds<T, WIDE>::kSym, kMask = (1u << kSym) - 1;
    u32 first = e & kMask, len = (e >> 8) & 31u;
    if (WIDE && len == 0) { const u32 a = pairs_one(L, t, win); first = a & 15u; len = a >> 4; }
    const u32 rest = PairsStrings<T, WIDE>::next(L, wave, t, p + len), f = L.lut[t][rest >> (32 - kBits)];
    u32 second = f & kMask, l2 = (f >> 8) & 31u;
    if ((f & kPairEscape) == 0) l2 = l2 ? L.len[t][second] : 0u;              // (length 0: a prefix that starts no code)
    else if (WIDE && l2 == 0) { const u32 b = pairs_one(L, t, rest); second = b & 15u; l2 = b >> 4; }
    return first | second << kSym | (len + l2) << 8;
}

// x << and x + the second byte of e, in one instruction each (the compiler takes two or three).
__device__ __forceinline__ u32 shl_byte1(u32 x, u32 e) {
    u32 r;
    asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_1 src1_sel:DWORD" : "=v"(r) : "v"(e), "v"(x));
    return r;
}
__device__ __forceinline__ u32 add_byte1(u32 x, u32 e) {
    u32 r;
    asm("v_add_u32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_1" : "=v"(r) : "v"(x), "v"(e));
    return r;
}

// The next 4 symbols of every blob: their representatives, and the positions behind them.  Written step by step across the
// blobs, so that the T look-ups of a step are in flight together.
template <int T, bool WIDE>
__device__ __forceinline__ void pairs_symbols(const PairsLds<T, WIDE>& L, u32 wave, PairsStrings<T, WIDE>& S, lc_f32x2 (&rep)[2][T]) {
    constexpr u32 kBits = PairsLds<T, WIDE>::kBits;
    u32 win[T], e[2][T];
#pragma unroll
    for (int t = 0; t < T; ++t) win[t] = PairsStrings<T, WIDE>::next(L, wave, t, S.p[t]);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        u32 escapes = 0;
#pragma unroll
        for (int t = 0; t < T; ++t) {
            e[h][t] = L.lut[t][win[t] >> (32 - kBits)];
            asm("" : "+v"(e[h][t]));             // keep it a 32-bit value (no 16-bit shift plus re-extension)
        }
#pragma unroll
        for (int t = 0; t < T; ++t) escapes |= e[h][t];
        if (__any((escapes & kPairEscape) != 0)) {
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const bool slow = (e[h][t] & kPairEscape) != 0;
                if (slow) e[h][t] = pairs_slow(L, wave, t, S.p[t], win[t], e[h][t]);
                const u32 p = add_byte1(S.p[t], e[h][t]);
                if (h == 0) win[t] = slow ? PairsStrings<T, WIDE>::next(L, wave, t, p) : shl_byte1(win[t], e[h][t]);
                S.p[t] = p;
            }
        } else {
#pragma unroll
            for (int t = 0; t < T; ++t) {
                if (h == 0) win[t] = shl_byte1(win[t], e[h][t]);
                S.p[t] = add_byte1(S.p[t], e[h][t]);
            }
        }
    }
#pragma unroll
    for (int t = 0; t < T; ++t) {
        rep[0][t] = L.rep[t][e[0][t] & 0xFFu];
        rep[1][t] = L.rep[t][e[1][t] & 0xFFu];
    }
}

// A row's 4 elements and 4 symbols of every blob: the additions, in blob order.
template <int T, int DT>
__device__ __forceinline__ void pairs_add(float (&x)[4], const lc_f32x2 (&rep)[2][T]) {
#pragma unroll
    for (int t = 0; t < T; ++t) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            x[2 * h] = __fadd_rn(x[2 * h], rep[h][t].x); x[2 * h + 1] = __fadd_rn(x[2 * h + 1], rep[h][t].y);
            if constexpr (DT != kF32) {          // (the running value as it reads back after a store)
                const u32 u = narrow16_pair(x[2 * h], x[2 * h + 1], DT == kBF16);
                x[2 * h] = widen16(u & 0xFFFFu, DT == kBF16); x[2 * h + 1] = widen16(u >> 16, DT == kBF16);
            }
        }
    }
}

// (plain stores: 957 us for 932)
template <int DT>
__device__ __forceinline__ void pairs_store(void* w_ref, u64 idx, const float (&x)[4]) {
    if constexpr (DT == kF32) __builtin_nontemporal_store(f32x4{x[0], x[1], x[2], x[3]}, reinterpret_cast<f32x4_any*>(static_cast<float*>(w_ref) + idx));
    else *reinterpret_cast<u32x2_any*>(static_cast<uint16_t*>(w_ref) + idx) =
             u32x2{narrow16_pair(x[0], x[1], DT == kBF16), narrow16_pair(x[2], x[3], DT == kBF16)};
}

// off: the chunk's entries of blob t's offset table in lane t (its start) and lane kMaxMany + t (its end); lane_bits: the lane
// lengths of its records; take, lengths: take the next chunk and ask for its entries, then for its lane lengths; each is called at
// most once, where its loads cost no wait, and of a chunk that is decoded late, so that it is a wavefront soon free that takes it
template <int T, bool WIDE, int DT, typename Take, typename Lengths>
__device__ __forceinline__ void pairs_chunk(PairsLds<T, WIDE>& L, u32 wave, void* __restrict__ w_ref, u64 n, Workspace* ws, HostResult* host,
                                            u32 c, u32 nchunks, u32 off, const u32 (&lane_bits)[T], u32 turns, u32 row_bits, u64 epoch, Take& take, Lengths& lengths) {
    typedef PairsLds<T, WIDE> Lds;
    typedef typename Raw<DT>::type RowT;
    const u32 lane = lane_id();
    PairsStrings<T, WIDE> S;
    const bool last = c + 1 == nchunks;
    bool loud = n - (u64)c * kChunk < kChunk;                // (a ragged chunk's lanes are not alike)
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const u32 o0 = read_lane(off, t), o1 = read_lane(off, kMaxMany + t);
        S.gw[t] = reinterpret_cast<const u32*>(uniform_ptr(L.rec_base[t]) + 4 * (u64)o0 + 2 * kW);
        S.nw[t] = o1 - o0 - kLaneBitsWords;               // >= 1 (validated)
        loud = loud || L.zero_bits[t] == 0 || lane_bits[t] != L.zero_bits[t];
    }
    const bool quiet = !__any(loud);
    if (quiet) {
        // every lane has the length of merged symbols only (see zero_chunk_bits); if so, nothing changes and w_ref is not read
        // (a payload of zero_bits per lane: a multiple of 512 words, the first of all blobs asked for at once; a word of one blob
        // after the other, 5 blobs of a sparse update of 2^27 elements 200 us; chunks taken as below and so, 138)
        typedef typename PairsWords<T, WIDE>::vec_any vec_any;
        u32x4 x[T][2], any = {0, 0, 0, 0};
        take();
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (u32 h = 0; h < 2; ++h) x[t][h] = *reinterpret_cast<const vec_any*>(S.gw[t] + 4 * (h * kW + lane));
        lengths();
#pragma unroll
        for (int t = 0; t < T; ++t) any |= x[t][0] | x[t][1];
#pragma unroll
        for (int t = 0; t < T; ++t)
            for (u32 i = 4 * (2 * kW + lane); i < S.nw[t]; i += 4 * kW) any |= *reinterpret_cast<const vec_any*>(S.gw[t] + i);
        if (!__any((any.x | any.y | any.z | any.w) != 0)) return;
    }
    u32 end[T];                                              // where the lane's strings end
    {
        PairsWords<T, WIDE> F[T];
#pragma unroll
        for (int t = 0; t < T; ++t) {
            end[t] = 31 + wave_incl_scan(lane_bits[t]);
            S.p[t] = end[t] - lane_bits[t];
            S.from[t] = 0;
            F[t].fetch(S, t, last);
        }
#pragma unroll
        for (int t = 0; t < T; ++t) F[t].place(S, L, wave, t);
    }
    // The windows move on, up to `turns` of them every 4 rows: those of blob `turn` and the next ones', unless they will do until
    // the blob's next turn.  The words are asked for 4 rows before they are put in place.
    constexpr u32 kMost = Lds::kWords * 32 - 1 - Lds::kStepBits;
    PairsWords<T, WIDE> F[Lds::kTurns];
    u32 turn = 0, asked = 0;
    auto place_words = [&]() {
#pragma unroll
        for (u32 i = 0; i < Lds::kTurns; ++i)
#pragma unroll
            for (int t = 0; t < T; ++t)
                if ((asked >> i & 1u) != 0 && (turn + i) % T == (u32)t) F[i].place(S, L, wave, t);
    };
    auto ask_for_words = [&](u32 rows_left) {
        turn = (turn + turns) % T;
        asked = 0;
        const u32 until = min(rows_left, 4 * (T + turns - 1) / turns + 4) * row_bits / 16, enough = until < kMost ? kMost - until : 0;
#pragma unroll
        for (u32 i = 0; i < Lds::kTurns; ++i)
#pragma unroll
            for (int t = 0; t < T; ++t)
                if (i < turns && (turn + i) % T == (u32)t && __any(S.p[t] > enough)) { asked |= 1u << i; F[i].fetch(S, t, last); }
    };
    // ... and at once, where a lane may run out of words within the next two rows
    auto have_words = [&]() {
        u32 most = 0;
#pragma unroll
        for (int t = 0; t < T; ++t) most = max(most, S.p[t]);
        if (!__any(most > kMost)) return;
#pragma unroll
        for (int t = 0; t < T; ++t)
            if (__any(S.p[t] > kMost)) { PairsWords<T, WIDE> now; now.fetch(S, t, last); now.place(S, L, wave, t); }
    };
    const u64 base = (u64)c * kChunk + lane * kV, left = n - (u64)c * kChunk;
    const u32 rows = left < kChunk ? (u32)left / kRowElems : kR;
    auto row = [&](const RowT& raw, u32 r) {
        float x[4];
        lc_f32x2 rep[2][T];
        unpack<DT>(raw, x);
        pairs_symbols(L, wave, S, rep);
        pairs_add<T, DT>(x, rep);
        pairs_store<DT>(w_ref, base + (u64)r * kRowElems, x);
    };
    // 8 to 12 rows are on their way ahead of the one being decoded
    constexpr u32 PF = 4;
    RowT A[PF], B[PF], C[PF];
    auto fetch = [&](RowT (&X)[PF], u32 at) {
#pragma unroll
        for (u32 k = 0; k < PF; ++k) X[k] = load_raw_any<DT>(w_ref, base + (u64)(at + k) * kRowElems);
    };
    const u32 whole = rows / PF * PF;
    // (of equally dense chunks the first four wavefronts take theirs first, one on each SIMD: few chunks to a wavefront, bf16, 16
    // symbols, 3 blobs of 2,926 chunks 145 us the call, in any order 148)
    const u32 early = wave < kPairsWaves / 2 ? kR / 2 - 2 * PF : kR / 2;
    u32 r = 0;
    if (whole > 0) fetch(A, 0);
    if (whole > PF) fetch(B, PF);
#pragma unroll 1
    for (; r < whole; r += PF) {
        place_words();                                       // (ahead of the rows, whose loads it would wait for)
        ask_for_words(rows - r);
        if (r == early && !quiet) take();
        if (r == kR / 2 + 4 * PF && !quiet) lengths();
        if (r + 2 * PF < whole) fetch(C, r + 2 * PF);
#pragma unroll
        for (u32 k = 0; k < PF; k += 2) {
            have_words();
            row(A[k], r + k);
            row(A[k + 1], r + k + 1);
        }
#pragma unroll
        for (u32 k = 0; k < PF; ++k) { A[k] = B[k]; B[k] = C[k]; }
    }
#pragma unroll 1
    for (; r < rows; ++r) { have_words(); row(load_raw_any<DT>(w_ref, base + (u64)r * kRowElems), r); }
    if (rows < kR) {
        // what is left of a ragged chunk, element by element
        have_words();
#pragma unroll 1
        for (u32 v = 0; v < kV; ++v) {
            const u64 i = base + (u64)rows * kRowElems + v;
            if (i >= n) continue;
            float x = load_one<DT>(w_ref, i);
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const u32 e = pairs_one(L, t, PairsStrings<T, WIDE>::next(L, wave, t, S.p[t]));
                S.p[t] += e >> 4;
                x = stored<DT>(__fadd_rn(x, L.rep[t][e & 15u].x));
            }
            store_one<DT>(w_ref, i, x);
        }
    }
    bool bad = false;
#pragma unroll
    for (int t = 0; t < T; ++t) bad = bad || S.p[t] + 32 * S.from[t] != end[t];
    if (__any(bad) && lane == 0) raise_status(ws, host, epoch, 4u);
}

// turns: windows that may move on every 4 rows, of a blob each; row_bits: 16 times the bits that a lane takes per row, at most
template <int T, bool WIDE, int DT>
__global__ __launch_bounds__(kPairsWaves * kW, T > 4 || WIDE ? 2 : 4) void k_decode_pairs(BlobList blobs, u32 first, void* __restrict__ w_ref, u64 n,
                                                     Workspace* ws, u32 nchunks, u64 epoch, HostResult* host, u32 turns, u32 row_bits) {
    typedef PairsLds<T, WIDE> Lds;
    __shared__ Lds L;
    const u32 tid = threadIdx.x, lane = tid & (kW - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (tid == 0) L.taken = kPairsWaves;
    if (tid == 0) L.stop = (__hip_atomic_load(&ws->dec_status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> 8) == epoch;
    __syncthreads();
    if (L.stop) return;                                  // a check found something: touch nothing
    static_assert(kMaxMany <= (int)kPairsWaves, "a wavefront per blob");
    if (wave < T) {
        const u32 t = wave;
        const DecSet& D = ws->dec_set[first + t];
        const u32 K = D.info.K, len = lane < kMaxSym ? D.info.len[lane] : 0u, code = lane < kMaxSym ? D.info.code[lane] : 0u;
        const u32 rep = lane < K ? D.info.rep_bits[lane & (kMaxSym - 1)] : 0x80000000u;
        const u32 coded = (u32)__popcll(__ballot(len != 0));
        u32x4 m[4];                                          // the tables of all the whole codes of 10 bits: entries 4 (64 k + lane) and on
#pragma unroll
        for (u32 k = 0; k < 4; ++k) m[k] = reinterpret_cast<const u32x4*>(D.multi)[k * kW + lane];
        if (lane == 0) {
            const uint8_t* blob = blobs.p[first + t];
            L.zero_bits[t] = zero_chunk_bits(read_lane(len, K), read_lane(code, K));
            L.rec_base[t] = blob + D.info.area;
            L.off_tab[t] = reinterpret_cast<const u32*>(blob + kHeaderBytes);
            L.nranks[t] = coded; L.merged[t] = K;
        }
        // the first two symbols of `bits`, which start with entry e's 10
        auto entry = [&](u32 e, u32 bits) {
            const u32 s0 = e & 15u, L0 = gather_lane(len, s0);
            u32 count = e >> 28, s1 = (e >> 4) & 15u;
            if (WIDE) {
                const u32 rest = (bits << L0) & ((1u << Lds::kBits) - 1), e1 = D.multi[rest >> (Lds::kBits - kMultiBits)];
                const u32 l1 = gather_lane(len, e1 & 15u);
                if (count == 1 && e1 != 0 && ((e1 >> 24) & 15u) != 0 && L0 + l1 <= Lds::kBits) { count = 2; s1 = e1 & 15u; }
            }
            const u32 both = L0 + gather_lane(len, s1);
            const bool none = e != 0 && ((e >> 24) & 15u) == 0;           // a prefix that starts no code
            return none ? K | K << Lds::kSym : count >= 2 ? s0 | s1 << Lds::kSym | both << 8 : count == 1 ? kPairEscape | s0 | L0 << 8 : kPairEscape;
        };
#pragma unroll
        for (u32 k = 0; k < 4; ++k) {
            const u32 i = 4 * (k * kW + lane), e[4] = {m[k].x, m[k].y, m[k].z, m[k].w};
            if constexpr (!WIDE) {
                reinterpret_cast<u32x2*>(L.lut[t])[k * kW + lane] = u32x2{entry(e[0], i) | entry(e[1], i + 1) << 16, entry(e[2], i + 2) | entry(e[3], i + 3) << 16};
            } else {
                u32 two[4];
#pragma unroll
                for (u32 j = 0; j < 4; ++j) two[j] = entry(e[j], 2 * (i + j)) | entry(e[j], 2 * (i + j) + 1) << 16;
                reinterpret_cast<u32x4*>(L.lut[t])[k * kW + lane] = u32x4{two[0], two[1], two[2], two[3]};
            }
        }
#pragma unroll
        for (u32 i = lane; i < Lds::kSyms * Lds::kSyms; i += kW)
            L.rep[t][i] = lc_f32x2{__uint_as_float(gather_lane(rep, i & (Lds::kSyms - 1))), __uint_as_float(gather_lane(rep, i >> Lds::kSym))};
        // a symbol's rank in canonical order (shorter codes first, then by index)
        const u32 place = lane < kMaxSym && len ? len * kMaxSym + lane : 0xFFFFu;
        u32 rank = 0;
        for (u32 j = 0; j < Lds::kSyms; ++j) rank += read_lane(place, j) < place ? 1u : 0u;
        if (lane < Lds::kSyms) L.len[t][lane] = len;
        if (lane >= coded && lane < Lds::kSyms) L.lj[t][lane] = 0xFFFFFFFFu;
        if (lane < Lds::kSyms && len) { L.lj[t][rank] = code << (32 - len); L.e_rank[t][rank] = (len << 4) | lane; }
    }
    __syncthreads();
    // A workgroup's wavefronts take its chunks as they come to them: what a chunk costs differs a lot where some hold merged symbols
    // only (dealt out in advance, 8 blobs of a sparse update of 2^27 elements 273 us, of 2^28 416; so, 186 and 252; of equally dense
    // chunks the same to 1 %).  One is taken halfway through the chunk before it (taken as that one began, 2^27 elements in layers
    // off alignment, of whose chunks a third is dense, 2 and 4 blobs 119 and 143 us, 103 and 120 so; 8 blobs 222 in advance, 187 so).
    auto chunk = [&](u32 k) { return blockIdx.x + gridDim.x * k; };         // (few chunks: on as many compute units as there are)
    auto offsets = [&](u32 c) {
        const u32 which = lane & (kMaxMany - 1);
        return lane < 2 * kMaxMany && which < T && c < nchunks ? L.off_tab[which][c + lane / kMaxMany] : 0u;
    };
    auto lengths = [&](u32 c, u32 off, u32 (&lane_bits)[T]) {
        if (c >= nchunks) return;
#pragma unroll
        for (int t = 0; t < T; ++t) lane_bits[t] = reinterpret_cast<const uint16_t*>(uniform_ptr(L.rec_base[t]) + 4 * (u64)read_lane(off, t))[lane];
    };
    u32 c = chunk(wave);                                    // (at most 2^18 chunks, and 8 more takings than those per workgroup)
    u32 off = offsets(c), bits[T] = {};
    lengths(c, off, bits);
    while (c < nchunks) {
        u32 after = 0, next = 0, next_bits[T] = {};
        bool taken = false, have = false;
        auto take = [&]() {
            u32 k = 0;
            if (lane == 0) k = atomicAdd(&L.taken, 1u);
            after = chunk(__builtin_amdgcn_readfirstlane(k));
            next = offsets(after);
            taken = true;
        };
        auto its_lengths = [&]() { lengths(after, next, next_bits); have = true; };
        pairs_chunk<T, WIDE, DT>(L, wave, w_ref, n, ws, host, c, nchunks, off, bits, turns, row_bits, epoch, take, its_lengths);
        if (!taken) take();
        if (!have) its_lengths();
#pragma unroll
        for (int t = 0; t < T; ++t) bits[t] = next_bits[t];
        off = next;
        c = after;
    }
}
// ----------------------------------------------------------------------------- launchers
void launch_batch_decode(const BatchDecArgs& a, const Tuning& tune, hipStream_t s) {
    hipLaunchKernelGGL(kb_dec_tables, dim3(a.count), dim3(256), 0, s, a);
    if (a.total_chunks) {
        hipLaunchKernelGGL(kb_dec_chunks, dim3((a.total_chunks + 3) / 4), dim3(256), 0, s, a);
        // single-wavefront workgroups, three to four times as many as the compute units hold at once (10 each, by their LDS)
        // as long as there are chunks for them: workgroups that draw cheap chunks (nothing but merged symbols) make
        // room for the next, which evens out the load better than a fixed deal of chunks to resident wavefronts
        // (40 tensors of 2^28 elements, 12 / 20 / 36 / 60 per unit: 520, 451, 444, 441 us at 4 bits, 103, 89, 84, 82 at 2)
        u32 waves = (u32)tune.num_cu * (u32)tune.decode_blocks_per_cu * 4u;
        if (waves > a.total_chunks) waves = a.total_chunks;
        if (a.dtype == kBF16) hipLaunchKernelGGL(kb_decode<kBF16>, dim3(waves), dim3(64), 0, s, a);
        else if (a.dtype == kF16) hipLaunchKernelGGL(kb_decode<kF16>, dim3(waves), dim3(64), 0, s, a);
        else hipLaunchKernelGGL(kb_decode<kF32>, dim3(waves), dim3(64), 0, s, a);
    }
}

void launch_dec_check(const BlobList& blobs, int first, int count, uint64_t n, int dtype, uint64_t max_total, Workspace* ws,
                      uint64_t epoch, HostResult* host, hipStream_t s) {
    const u64 nchunks = num_chunks_of(n);
    // one chunk per wavefront while that is at most a few rounds of workgroups on the chip, else four
    const bool four = (u64)count * ((nchunks + 3) / 4) > 8192;
    const u64 per_block = four ? 16 : 4;
    const u64 blocks = nchunks ? (nchunks + per_block - 1) / per_block : 1;
    if (four) hipLaunchKernelGGL(k_dec_check<4>, dim3((u32)blocks, (u32)count), dim3(256), 0, s, blobs, (u32)first, (u64)n, (u64)max_total,
                                 ws, (u32)nchunks, (u64)epoch, host, (u32)dtype);
    else hipLaunchKernelGGL(k_dec_check<1>, dim3((u32)blocks, (u32)count), dim3(256), 0, s, blobs, (u32)first, (u64)n, (u64)max_total,
                            ws, (u32)nchunks, (u64)epoch, host, (u32)dtype);
}



template <int T, bool WIDE>
static void launch_pairs_t(const BlobList& blobs, int first, void* w_ref, uint64_t n, int dtype, Workspace* ws, uint64_t epoch,
                           HostResult* host, u32 cus, u32 turns, u32 row_bits, hipStream_t s) {
    static_assert(sizeof(PairsLds<T, WIDE>) <= kLdsPerCu, "a workgroup fits a compute unit");
    // (two workgroups of up to 4 blobs that keep at most 7 buckets share a compute unit by their LDS and registers)
    const u64 need = num_chunks_of(n), cap = (u64)cus * (2 * sizeof(PairsLds<T, WIDE>) + 2 * 1280 <= kLdsPerCu ? 2 : 1);
    const dim3 grid((u32)(need < cap ? need : cap)), wg(kPairsWaves * kW);
#define LC_PAIRS(DT) hipLaunchKernelGGL((k_decode_pairs<T, WIDE, DT>), grid, wg, 0, s, blobs, (u32)first, w_ref, (u64)n, ws, (u32)num_chunks_of(n), (u64)epoch, host, turns, row_bits)
    if (dtype == kBF16) LC_PAIRS(kBF16);
    else if (dtype == kF16) LC_PAIRS(kF16);
    else LC_PAIRS(kF32);
#undef LC_PAIRS
}

void launch_decode_pairs(const BlobList& blobs, int first, int count, void* w_ref, uint64_t n, int dtype, Workspace* ws,
                         uint64_t epoch, HostResult* host, double row_bits, bool wide, const Tuning& tune, hipStream_t s) {
    if (n == 0) return;
    // A window's turn comes every 4 T / turns rows, with words as of 4 rows before: its strings should take no more than some
    // 170 (wide: 350) bits in that time.  (the fullest lane: some 15 % more than the average, and half a bit)
    const double full = 1.15 * row_bits + 0.5, room = (wide ? 350 : 170) / full / 4 - 1;
    const u32 turns = count <= room ? 1 : count <= 2 * room || count <= 4 ? 2 : 4, bits16 = (u32)(16 * full);
#define LC_PAIRS(T, W) launch_pairs_t<T, W>(blobs, first, w_ref, n, dtype, ws, epoch, host, (u32)tune.num_cu, turns, bits16, s)
    switch (count) {
        case 2: if (wide) LC_PAIRS(2, true); else LC_PAIRS(2, false); break;
        case 3: if (wide) LC_PAIRS(3, true); else LC_PAIRS(3, false); break;
        case 4: if (wide) LC_PAIRS(4, true); else LC_PAIRS(4, false); break;
        case 5: LC_PAIRS(5, false); break;
        case 6: LC_PAIRS(6, false); break;
        case 7: LC_PAIRS(7, false); break;
        case 8: LC_PAIRS(8, false); break;
    }
#undef LC_PAIRS
}

template <int T, int DT>
static void launch_fused_td(const BlobList& blobs, int first, void* w_ref, uint64_t n, Workspace* ws, uint64_t epoch,
                            HostResult* host, u32 blocks, u32 pay_words, bool long_codes, hipStream_t s) {
    const size_t lds = 4 * (size_t)(pay_words + kFusedSlack);
    if (long_codes) hipLaunchKernelGGL((k_decode_fused<T, true, DT>), dim3(blocks), dim3(64), lds, s, blobs, (u32)first, w_ref,
                                       (u64)n, ws, (u32)num_chunks_of(n), (u64)epoch, host, pay_words);
    else hipLaunchKernelGGL((k_decode_fused<T, false, DT>), dim3(blocks), dim3(64), lds, s, blobs, (u32)first, w_ref,
                            (u64)n, ws, (u32)num_chunks_of(n), (u64)epoch, host, pay_words);
}

template <int T>
static void launch_fused_t(const BlobList& blobs, int first, void* w_ref, uint64_t n, int dtype, Workspace* ws, uint64_t epoch,
                           HostResult* host, u32 blocks, u32 pay_words, bool long_codes, hipStream_t s) {
    if (dtype == kBF16) launch_fused_td<T, kBF16>(blobs, first, w_ref, n, ws, epoch, host, blocks, pay_words, long_codes, s);
    else if (dtype == kF16) launch_fused_td<T, kF16>(blobs, first, w_ref, n, ws, epoch, host, blocks, pay_words, long_codes, s);
    else launch_fused_td<T, kF32>(blobs, first, w_ref, n, ws, epoch, host, blocks, pay_words, long_codes, s);
}

size_t fused_lds_bytes(int count, uint32_t pay_words) {
    static const size_t head[kMaxMany] = {sizeof(FusedHead<1>), sizeof(FusedHead<2>), sizeof(FusedHead<3>), sizeof(FusedHead<4>),
                                          sizeof(FusedHead<5>), sizeof(FusedHead<6>), sizeof(FusedHead<7>), sizeof(FusedHead<8>)};
    return head[count - 1] + 4 * (size_t)(pay_words + kFusedSlack);
}

void launch_decode_fused(const BlobList& blobs, int first, int count, void* w_ref, uint64_t n, int dtype, Workspace* ws,
                         uint64_t epoch, HostResult* host, uint32_t pay_words, bool long_codes, const Tuning& tune,
                         hipStream_t s) {
    const u64 nchunks = num_chunks_of(n);
    if (nchunks == 0) return;
    // one wavefront per workgroup; as many workgroups per compute unit as their LDS areas allow
    u64 per_cu = kLdsPerCu / fused_lds_bytes(count, pay_words);
    if (per_cu > (u64)tune.fused_waves_per_cu) per_cu = tune.fused_waves_per_cu;
    if (per_cu < 1) per_cu = 1;
    u64 blocks = (u64)tune.num_cu * per_cu;
    if (blocks > nchunks) blocks = nchunks;
    const u32 b = (u32)blocks;
    switch (count) {
        case 1: launch_fused_t<1>(blobs, first, w_ref, n, dtype, ws, epoch, host, b, pay_words, long_codes, s); break;
        case 2: launch_fused_t<2>(blobs, first, w_ref, n, dtype, ws, epoch, host, b, pay_words, long_codes, s); break;
        case 3: launch_fused_t<3>(blobs, first, w_ref, n, dtype, ws, epoch, host, b, pay_words, long_codes, s); break;
        case 4: launch_fused_t<4>(blobs, first, w_ref, n, dtype, ws, epoch, host, b, pay_words, long_codes, s); break;
        case 5: launch_fused_t<5>(blobs, first, w_ref, n, dtype, ws, epoch, host, b, pay_words, long_codes, s); break;
        case 6: launch_fused_t<6>(blobs, first, w_ref, n, dtype, ws, epoch, host, b, pay_words, long_codes, s); break;
        case 7: launch_fused_t<7>(blobs, first, w_ref, n, dtype, ws, epoch, host, b, pay_words, long_codes, s); break;
        default: launch_fused_t<8>(blobs, first, w_ref, n, dtype, ws, epoch, host, b, pay_words, long_codes, s); break;
    }
}

// w_ref null: the verifying sweep (nothing but the blob is read)
void launch_decode(const uint8_t* blob, void* w_ref, uint64_t n, int dtype, Workspace* ws, int set, uint64_t epoch, HostResult* host,
                   const Tuning& tune, hipStream_t s) {
    const u64 nchunks = num_chunks_of(n);
    if (nchunks == 0) return;
    const bool verify = w_ref == nullptr;
    // Up to so many chunks per compute unit the grid is just what 3 workgroups of it hold by their LDS (decode_blocks_per_cu has
    // no say): a wavefront then looks ahead to its next chunk, and no second round of workgroups pays its start.  Above,
    // smaller shares even out chunks of unlike cost, and only 2 workgroups share a unit, by the size of their payload
    // areas: a sweep that reads and writes runs better on fewer streams.  Where the one passes the other depends on the
    // bytes of a row and on what the chunks hold; few / many, us, fp32: 7,000 chunks dense 212 / 199, layered 176 / 152,
    // sparse 31 / 31; 8,445 236 / 238, 176 / 155, 29 / 32; 16,384 441 / 423, 295 / 258, 32 / 35.  bf16, dense: 8,192
    // 128 / 138, 16,384 228 / 243, 32,768 423 / 453, 49,152 661 / 719.  binary64: as far as rows are fetched a group
    // ahead, a chunk per wavefront and 2 workgroups per unit.  A verifying sweep only reads.
    const u64 few_per_cu = verify ? 48 : dtype == kF64 ? 8 : dtype == kF32 ? 24 : 256;
    const bool few = nchunks <= (u64)tune.num_cu * few_per_cu;
    const u64 blocks = balanced_workers((nchunks + 3) / 4, (u64)tune.num_cu * (few ? 3 : tune.decode_blocks_per_cu));
    const dim3 grid((u32)blocks), wg(256);
    const int ahead = few || dtype != kF64;
    const u32 pay_words = blocks <= (u64)tune.num_cu ? kPayWordsOne : few && blocks > 2 * (u64)tune.num_cu ? kPayWords : verify ? kPayWordsVerify : kPayWordsTwo;
    constexpr size_t fixed = sizeof(DecLds) + 4 * kRingWords * kW * 4, area = 4 * sizeof(uint4);
    static_assert(fixed + area * (kPayWordsOne / 4 + 1) <= kLdsPerCu && fixed + area * (kPayWordsTwo / 4 + 1) <= kLdsPerCu / 2 - 1280 &&
                  fixed + area * (kPayWords / 4 + 1) <= kLdsPerCu / 3 - 1280, "workgroups that share a compute unit (LDS is given in steps of 1280 bytes)");
    const size_t lds = area * (pay_words / 4 + 1);
    if (verify) {
        hipLaunchKernelGGL((k_decode<kF32, true>), grid, wg, lds, s, blob, (void*)nullptr, (u64)n, ws, (u32)nchunks, ahead, (u64)epoch, host, pay_words, (u32)set);
        return;
    }
#define LC_DECODE(DT) hipLaunchKernelGGL((k_decode<DT>), grid, wg, lds, s, blob, w_ref, (u64)n, ws, (u32)nchunks, ahead, (u64)epoch, host, pay_words, (u32)set)
    if (dtype == kF64) LC_DECODE(kF64);
    else if (dtype == kBF16) LC_DECODE(kBF16);
    else if (dtype == kF16) LC_DECODE(kF16);
    else LC_DECODE(kF32);
#undef LC_DECODE
}

}  // namespace lc
