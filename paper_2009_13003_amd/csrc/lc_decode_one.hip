// The restore of a short vector in one launch (gfx950, wave64): Algorithm 1 line 7; Section 3, C1.
#include "lc_meeting.h"

namespace lc {

// ----------------------------------------------------------------------------- k_decode_one
// The restore of a short vector in one launch: a workgroup of eight wavefronts per chunk, all of them resident together.
// With a wavefront per chunk most of the chip idles while each lane's string of 256 codes is taken apart step by step and
// its rows are restored behind that: 17.1 us at 2^20 fp32 elements, behind a check kernel of 6.4; all of it here 12.6 (whole calls,
// two kernels / one: see fits_in_one).  Here every workgroup checks
// the header and its chunk for itself and builds the tables in LDS; the workgroups meet (GridMeeting) between their findings
// and the first store, so that a blob that is refused leaves w_ref untouched, and the meeting's wait lies behind the decoding.
//
// A string is decoded in eight segments at once, one per wavefront: cut at eighths of its bits, each segment is
// first taken from its cut, in the middle of some code.  A prefix code falls into step with itself after a few codes, so
// where such a segment passes its end is mostly right; each is then taken again from where the one before it ended, until no
// start moves any more.  The first segment starts right, so after turn k the first k are right whatever the string, and
// mostly all are after two.  Then the segments' numbers of symbols are known, and a last turn notes the symbols in
// their places.  (A segment's end is the first code that starts at or behind the cut, so that it does not depend on the steps.)
constexpr u32 kSegs = 8, kOneDecThreads = kSegs * kW, kOneSegRows = kR / kSegs;
constexpr u32 kOnePayWords = kChunk * 15 / 32;               // the longest payload there is

struct OneDecLds {
    DecLds tab;
    uint8_t one[1u << kMultiBits];
    uint16_t ends[1u << kMultiBits];
    u32 hdr[kHeaderBytes / 4];
    alignas(16) u32 pay[kOnePayWords];
    u32 syms[kR * kV / 8][kW];           // 8 symbols of 4 bits per word: row k of lane l is in [k / 2][l]
    u32 end[kSegs][kW], count[kSegs][kW];
    u64 total0;
    u32 go, moved[kSegs + 1];            // (the last: some string is wrong)
    u32 set, few;                        // some bit of the payload is set; its kept symbols are in the notes
};

static_assert(2 * (sizeof(OneDecLds) + 1280) <= kLdsPerCu, "two workgroups per compute unit: the host counts on that many being resident");

// Several blobs of one vector (lc_decode_many): one after the other, the running values in registers; w_ref is read and written
// once, behind the one meeting.  Check, wait and fused sweep against this, us: 8 blobs of 2^20 fp32 elements at 3 bits 111.9 / 100.5,
// 3 of 2^17 at 4 bits 103 / 53, 12 of 2^19 bf16 at 4 bits 378 / 175, 8 of 2^22 binary64 295 / 122.  (The running values take
// binary64 to the 128 registers that two workgroups per compute unit leave: 20 spill, 52 bytes per lane, and in every type 42
// scalar ones to lanes of vector registers.)
struct OneDecArgs {
    BlobList blobs; void* w_ref; u64 n, max_total;
    Workspace* ws; HostResult* host; u64 epoch;
    u64 goal[kMeetLines];
    u32 count, nchunks, lines, limit;
};

// This lane's segment from bit `from` of its string to the first code that starts at `to` or behind: where that is, and how many
// symbols lie between.  NOTE: they go to the lane's column of `noted`, from symbol `at` on (never past its 256).  *bad: a prefix
// that starts no code.  LONG: some codes are longer than 10 bits.
constexpr u32 kNoCode = kMultiBits << 24;                    // the table's entry for one: no symbols
template <bool NOTE, bool LONG>
__device__ __forceinline__ u32 take_segment(const OneDecLds& L, u32 nwords, u32 first_bit, u32 from, u32 to,
                                            u32* noted, u32 at, u32* count, bool* bad) {
    constexpr u32 kStep = LONG ? 15 : kMultiBits;            // bits a step may take
    BitReader<true> br;
    br.start(L.pay, nwords, first_bit + from);
    u32 pos = from, i = at;
    bool none = false;
    auto look = [&](bool on) {
        u32 e = L.tab.multi[(u32)(br.win >> (64 - kMultiBits))];
        if (LONG && __any(on && e == 0)) { if (e == 0) e = decode_long(L.tab, br.win); }
        none = none || (on && e == kNoCode);
        return e;
    };
    auto take = [&](u32 sy, u32 len, u32 m) {
        if (NOTE) {
            const u64 s = (u64)sy << (4 * (i & 7));
            const u32 w = i >> 3;
            if (w < kR * kV / 8) atomicOr(&noted[w * kW], (u32)s);
            if ((s >> 32) != 0 && w + 1 < kR * kV / 8) atomicOr(&noted[(w + 1) * kW], (u32)(s >> 32));
        }
        i += m; pos += len;
        br.drop(len);
    };
    while (__any(pos + kStep <= to)) {                       // whole steps (33 valid bits take three of 10 or two of 15)
        br.refill();
#pragma unroll
        for (int rep = 0; rep < (LONG ? 2 : 3); ++rep) {
            const bool on = pos + kStep <= to;
            const u32 e = look(on), x = on ? e : 0u;
            take(x & 0xFFFFFFu, (x >> 24) & 15u, x >> 28);
        }
    }
    while (__any(pos < to)) {                                // the rest, up to the first code's end that is not before `to`
        br.refill();
        const bool on = pos < to;
        const u32 e = look(on), r = to - pos;
        const u32 ends = L.ends[(u32)(br.win >> (64 - kMultiBits))], m = on && r <= kMultiBits ? ends >> r : 0u;
        u32 len = (e >> 24) & 15u, k = e >> 28;
        if (m != 0) { len = r + (u32)__builtin_ctz(m); k = (u32)__builtin_popcount(ends & ((2u << len) - 1)); }
        if (!on) { len = 0; k = 0; }
        take(e & ((1u << (4 * k)) - 1), len, k);
    }
    *count = i - at; *bad = none;
    return pos;
}

// A chunk of few kept symbols, by one wavefront: each lane goes from one kept symbol of its string to the next (the merged symbol's
// code is `m` zero bits, shorter than any other: see decode_sparse) and notes them, place << 4 | symbol, in its column of `noted`.
// The codes are few enough to be compared with (key: code_key of lane j), so that such a chunk needs no tables.
// Returns how many, which may be more than the kFewNotes that are noted; *wrong: not `elems` symbols in `bits` bits.
constexpr u32 kFewNotes = kR * kV / 8, kFewEach = kFewNotes / kSegs;
__device__ __forceinline__ u32 take_few(const OneDecLds& L, u32 nwords, u32 first_bit, u32 bits, u32 elems, u32 m, u32 key, u32* noted, bool* wrong) {
    BitReader<true> br;
    br.start(L.pay, nwords, first_bit);
    const u32 wi0 = br.wi, avail0 = br.avail, inv = 65536u / m + 1;         // (z inv >> 16 = z / m for z <= 32, m <= 15)
    u32 pos = 0, count = 0;
    bool none = false;
    br.refill();
    while (__any(pos < elems)) {
        const u32 top = (u32)(br.win >> 32), zeros = top != 0 ? (u32)__builtin_clz(top) : 32u;
        const u32 run = min(zeros * inv >> 16, elems - pos);
        pos += run;
        br.drop(run * m);
        br.refill();
        const bool kept = pos < elems && (u32)(br.win >> (64 - m)) != 0;
        if (__any(kept)) {
            const u32 at = (u32)(br.win >> (64 - 15)) << 8 | 0xFFu;
            u32 best = 0;
#pragma unroll
            for (u32 j = 0; j < kMaxSym; ++j) { const u32 kj = read_lane(key, j); best = max(best, kj <= at ? kj : 0u); }
            const u32 len = (best >> 4) & 15u;
            if (kept) {
                none = none || len == 0 || (at >> 8) >= (best >> 8) + (0x8000u >> len);      // starts no code
                if (count < kFewNotes) noted[count * kW] = (pos << 4) | (best & 15u);
                ++count;
                pos = none ? elems : pos + 1;
                br.drop(len);
            }
            br.refill();
        }
    }
    *wrong = none || avail0 + 32 * (br.wi - wi0) - br.avail != bits;
    return count;
}

// x + the representative, as the parameters' type holds it (16-bit types: rounded after every blob)
template <int DT> __device__ __forceinline__ typename Val<DT>::type restored(typename Val<DT>::type x, typename Val<DT>::type rep) {
    if constexpr (DT == kF64) return add_rn(x, rep);
    else return stored<DT>(add_rn(x, rep));
}

// MANY: more than one blob.
template <int DT, bool MANY>
__global__ __launch_bounds__(kOneDecThreads, 4) void k_decode_one(OneDecArgs a) {
    typedef typename Val<DT>::type val_t;
    __shared__ OneDecLds L;
    const u32 t = threadIdx.x, lane = lane_id(), v = __builtin_amdgcn_readfirstlane(t >> 6), c = blockIdx.x;
    const u64 n = a.n, base = (u64)c * kChunk;
    GridMeeting meet = {a.ws->meeting(), 0, a.lines, a.limit};
#pragma unroll
    for (u32 k = 0; k < kMeetLines; ++k) meet.goal = lane == k ? a.goal[k] : meet.goal;
    // this wavefront's 8 rows of w_ref, and which of them hold a kept symbol
    val_t x[kOneSegRows][kV];
    u32 keeps = 0;
    auto row = [&](u32 k) { return base + (u64)(v * kOneSegRows + k) * kRowElems; };
    // (binary64: plain loads, two of which share their lines: 2^22 elements in layers 44.1 -> 42.5 us the call)
    auto fetch = [&](u32 k) {
        if (row(k) + kRowElems <= n) load_row_any<DT, DT != kF64>(a.w_ref, row(k) + lane * kV, x[k]);
        else load_row_v<DT>(a.w_ref, row(k) + lane * kV, n, x[k]);
    };
    if (MANY) {
#pragma unroll
        for (u32 k = 0; k < kOneSegRows; ++k) fetch(k);
    }
    const u32 elems = n - base < kChunk ? (u32)(n - base) : kChunk, tail = elems % kRowElems;
    const u32 mine = elems / kRowElems * kV + (tail > lane * kV ? min(tail - lane * kV, kV) : 0u);
    const u64 area = chunk_area_of(a.nchunks);
    bool refuse = false;                                     // (the same in every thread)
#pragma unroll 1
    for (u32 b = 0; b < (MANY ? a.count : 1u); ++b) {
        const uint8_t* blob = a.blobs.p[b];
        const bool last = !MANY || b + 1 == a.count;
        if (MANY && b) __syncthreads();                      // (everyone is through with the blob before)
        if (t < kHeaderBytes / 4) L.hdr[t] = reinterpret_cast<const u32*>(blob)[t];
        for (u32 i = t; i < kR * kV / 8 * kW; i += kOneDecThreads) L.syms[0][i] = 0;
        if (t < kSegs + 1) L.moved[t] = 0;
        if (t == 0) L.set = 0;
        __syncthreads();
        // ---- the header: every workgroup comes to the same findings (as k_dec_check's)
        const u32* hdr = L.hdr;
        const u64 hn = hdr[2] | ((u64)hdr[3] << 32), total = hdr[10] | ((u64)hdr[11] << 32);
        const bool sound = hdr[0] == 0x3142434Cu && hdr[1] == (1u | (kHeaderBytes << 16)) && hdr[12] == 0;
        const bool head_ok = sound && hn == n && hdr[15] == (u32)DT && hdr[9] == a.nchunks && total >= area && total <= a.max_total && ((total - area) & 3) == 0;
        if (!head_ok) {
            // (a sound blob for another vector or element type: a bad argument)
            if (t == 0) {
                if (c == 0) { raise_status(a.ws, a.host, a.epoch, sound && (hn != n || hdr[15] != (u32)DT) ? 1u : 4u); a.host->bytes[0] = 0; }
                meet.arrive(2);
            }
            return;
        }
        const u64 tw = (total - area) / 4;
        const u32 K = hdr[5];
        // ---- this chunk's record: its place in the offset table, its lane lengths, its payload
        const u32* off_tab = reinterpret_cast<const u32*>(blob + kHeaderBytes);
        const u64 o0 = load_uniform(off_tab + c), o1 = load_uniform(off_tab + c + 1);
        bool ok = o0 <= o1 && o1 <= tw && o1 - o0 >= kLaneBitsWords && (c > 0 || o0 == 0) && (c + 1 < a.nchunks || o1 == tw);
        u32 bits = 0, nwords = 0, set = 0;
        if (ok) {
            typedef u32x4 __attribute__((aligned(4))) u32x4_word;
            const u32* rec = reinterpret_cast<const u32*>(blob + area) + o0;
            nwords = (u32)min(o1 - o0 - kLaneBitsWords, (u64)kOnePayWords);          // (more than that is refused below)
            bits = reinterpret_cast<const uint16_t*>(rec)[lane];
            const u32* from = rec + kLaneBitsWords;
            for (u32 i = t; i < nwords / 4; i += kOneDecThreads) {
                const u32x4 x = reinterpret_cast<const u32x4_word*>(from)[i];
                reinterpret_cast<u32x4*>(L.pay)[i] = x;
                set |= x.x | x.y | x.z | x.w;
            }
            if (t < (nwords & 3)) { const u32 x = from[nwords / 4 * 4 + t]; L.pay[nwords / 4 * 4 + t] = x; set |= x; }
        }
        const u32 incl = wave_incl_scan(bits), sum = read_lane(incl, kW - 1);
        ok = ok && o1 - o0 == kLaneBitsWords + ((sum + 31) >> 5) && sum > 0 && !__any(bits > kR * kV * 15);
        // ---- the symbols and their codes (by every wavefront: none waits for another's)
        DecSymbol sy = {0, 0, 0, 0};
        ok = dec_symbols(hdr, n, a.nchunks, tw, &sy) && ok;
        const u32 max_len = wave_max_u32(sy.len);
        if (v == 0) {
            if (lane < kMaxSym) {
                L.tab.rep[lane] = __uint_as_float(lane < K ? sy.rep : 0x80000000u);
                L.tab.rep64[lane] = lane < K ? __hiloint2double((int)sy.rep_hi, (int)sy.rep) : -0.0;
            }
            if (max_len > kMultiBits) build_longs(L.tab, sy.len, sy.code);
        }
        // The rows of w_ref are on their way while the strings are decoded; of a chunk of few kept symbols (see kSparseSlack)
        // only those that hold one, and only when that is known (2^23 fp32 elements, sparse: 28.4 us with all of them, 26.0 so).
        const u32 len_merged = read_lane(sy.len, K & 15u);
        const bool sparse = sum <= elems * len_merged + kSparseSlack;
        const bool late = !MANY && (DT == kF64 || sparse);   // (binary64: their registers would spill meanwhile)
        if (!MANY && !late) {
#pragma unroll
            for (u32 k = 0; k < kOneSegRows; ++k) fetch(k);
        }
        refuse = refuse || !ok;
        if (t == 0) {
            if (!ok) raise_status(a.ws, a.host, a.epoch, 4u);
            if (last || refuse) meet.arrive(2, refuse);      // (what is found from here on in this workgroup keeps only its own rows back)
        }
        if (refuse) return;
        // A chunk of merged symbols only, whose code is that of no bit set: so is every word of its payload, and nothing is left to
        // do.  (A restore that changes nothing, 512 chunks of fp32: 23.4 -> 17.8 us; 19.9 by k_dec_check and k_decode, which look
        // for such chunks too.)
        bool quiet = len_merged != 0 && read_lane(sy.code, K & 15u) == 0 && !__any(bits != mine * len_merged);
        if (quiet) {
            if (set != 0) L.set = 1;
            __syncthreads();
            quiet = L.set == 0;
        }
        // ... and one of few others.  (Heavy tails at 3 bits, 64 / 256 / 512 chunks: 22.6 / 23.0 / 25.0 -> 19.9 / 19.7 / 22.6 us;
        // 24.0 / 23.6 / 23.0 by the two kernels.)
        const u32 first_bit = incl - bits;
        bool few = !MANY && !quiet && sparse && len_merged != 0 && read_lane(sy.code, K & 15u) == 0 && !__any(bits > mine * len_merged + kSparseLaneSlack);
        if (few) {
            if (v == 0) {
                bool wrong;
                const u32 count = take_few(L, nwords, first_bit, bits, mine, len_merged, code_key(sy.len, sy.code), &L.syms[0][lane], &wrong);
                const bool noted = !__any(count > kFewNotes);
                L.count[0][lane] = count;
                if (noted && __any(wrong) && lane == 0) { L.moved[kSegs] = 1; raise_status(a.ws, a.host, a.epoch, 4u); }
                if (lane == 0) L.few = noted ? 1u : 0u;
            }
            __syncthreads();
            few = L.few != 0;
            if (!few) {                                      // (as if nothing had been noted)
                for (u32 i = t; i < kR * kV / 8 * kW; i += kOneDecThreads) L.syms[0][i] = 0;
            }
        }
        val_t few_x[kFewEach];
        u32 few_at[kFewEach], few_count = 0;
        if (few) {
            // note k of a lane is wavefront k mod 8's; its element is on its way while the workgroups meet
            few_count = L.count[0][lane];
#pragma unroll
            for (u32 k = 0; k < kFewEach; ++k) {
                few_at[k] = L.syms[v + kSegs * k][lane];
                const u32 p = few_at[k] >> 4;
                if (v + kSegs * k < few_count) few_x[k] = load_one_v<DT>(a.w_ref, base + (p / kV) * kRowElems + lane * kV + p % kV);
            }
        }
        u64 seen = last && v == 0 && (quiet || few) ? meet.look(2) : 0ull;
        if (!quiet && !few) {
            dec_build_multi<kOneDecThreads>(L.tab.multi, L.one, L.ends, kNoCode, sy.len, sy.code, t);
            __syncthreads();
            // ---- the string of every lane, a segment per wavefront
            const u32 cut = bits * v / kSegs, to = bits * (v + 1) / kSegs;
            const bool long_codes = max_len > kMultiBits;
            u32 start = cut, count = 0, end;
            bool bad = false;
            auto segment = [&]() {
                end = long_codes ? take_segment<false, true>(L, nwords, first_bit, start, to, nullptr, 0, &count, &bad)
                                 : take_segment<false, false>(L, nwords, first_bit, start, to, nullptr, 0, &count, &bad);
                L.end[v][lane] = end;
            };
            segment();
            __syncthreads();
#pragma unroll 1
            for (u32 turn = 0; turn < kSegs; ++turn) {           // (after turn k the first k + 2 segments are right)
                const u32 now = v ? L.end[v - 1][lane] : 0u;
                const bool moves = __any(now != start);
                __syncthreads();                                 // (everyone has read the ends)
                if (moves) {
                    start = now;
                    segment();
                    if (lane == 0) L.moved[turn] = 1;
                }
                __syncthreads();
                if (L.moved[turn] == 0) break;
            }
            L.count[v][lane] = count;
            __syncthreads();
            u32 before = 0, all = 0;
#pragma unroll
            for (u32 k = 0; k < kSegs; ++k) { const u32 m = L.count[k][lane]; before += k < v ? m : 0u; all += m; }
            // a string that does not hold its lane's symbols in exactly its stated length
            const bool wrong = bad || all != mine || (v == kSegs - 1 && end != bits);
            if (__any(wrong) && lane == 0) { L.moved[kSegs] = 1; raise_status(a.ws, a.host, a.epoch, 4u); }
            if (last && v == 0) seen = meet.look(2);             // (on its way meanwhile)
            if (long_codes) take_segment<true, true>(L, nwords, first_bit, start, to, &L.syms[0][lane], before, &count, &bad);
            else take_segment<true, false>(L, nwords, first_bit, start, to, &L.syms[0][lane], before, &count, &bad);
        }
        if (last && v == 0) { const bool met = meet.wait(2, seen); if (lane == 0) L.go = met ? 1u : 0u; }
        __syncthreads();
        if (L.moved[kSegs] != 0) {
            if (!last && t == 0) meet.arrive(2, true);
            return;
        }
        if (last && !L.go) return;
        if (c == 0 && t == 0) { a.host->max_len[b] = max_len; if (last || b) a.host->bytes[b] = total; }
        if (MANY && c == 0 && t == 0 && b == 0) L.total0 = total;        // (bytes[0] says that the workgroups met)
        if (quiet) continue;
        if (few) {
#pragma unroll
            for (u32 k = 0; k < kFewEach; ++k) {
                const u32 p = few_at[k] >> 4;
                if (v + kSegs * k < few_count)
                    store_one_v<DT>(a.w_ref, base + (p / kV) * kRowElems + lane * kV + p % kV, add_rn(few_x[k], L.tab.template rep_of<DT>(few_at[k] & 15u)));
            }
            continue;
        }
        // ---- Algorithm 1 line 7; a row without a kept symbol stays as it is
        u32 syms[kOneSegRows], here = 0;
#pragma unroll
        for (u32 k = 0; k < kOneSegRows; ++k) {
            syms[k] = (L.syms[(v * kOneSegRows + k) / 2][lane] >> (16 * (k & 1))) & 0xFFFFu;
            // (places behind the vector's end hold symbol 0: they are masked where they are stored)
            here |= __any(syms[k] != K * 0x1111u) ? 1u << k : 0u;
        }
        keeps |= here;
        if (late) {
#pragma unroll
            for (u32 k = 0; k < kOneSegRows; ++k) if ((here >> k) & 1u) fetch(k);
        }
#pragma unroll
        for (u32 k = 0; k < kOneSegRows; ++k) {
            if (((here >> k) & 1u) == 0) continue;
            if constexpr (MANY) {
#pragma unroll
                for (u32 e = 0; e < kV; ++e) {
                    const u32 one = (syms[k] >> (4 * e)) & 15u;
                    x[k][e] = one != K ? restored<DT>(x[k][e], L.tab.template rep_of<DT>(one)) : x[k][e];
                }
            } else {
#pragma unroll
                for (u32 e = 0; e < kV; ++e) x[k][e] = add_rn(x[k][e], L.tab.template rep_of<DT>((syms[k] >> (4 * e)) & 15u));
                if (row(k) + kRowElems <= n) store4_any<DT>(a.w_ref, row(k) + lane * kV, x[k]);
                else {
#pragma unroll
                    for (u32 e = 0; e < kV; ++e)
                        if (row(k) + lane * kV + e < n && ((syms[k] >> (4 * e)) & 15u) != K) store_one_v<DT>(a.w_ref, row(k) + lane * kV + e, x[k][e]);
                }
            }
        }
    }
    if (!MANY) return;
    if (c == 0 && t == 0) a.host->bytes[0] = L.total0;
#pragma unroll
    for (u32 k = 0; k < kOneSegRows; ++k) {
        if (((keeps >> k) & 1u) == 0) continue;
        if (row(k) + kRowElems <= n) store4_any<DT>(a.w_ref, row(k) + lane * kV, x[k]);
        else {
#pragma unroll
            for (u32 e = 0; e < kV; ++e)
                if (row(k) + lane * kV + e < n) store_one_v<DT>(a.w_ref, row(k) + lane * kV + e, x[k][e]);
        }
    }
}

void launch_decode_one(const BlobList& blobs, int count, void* w_ref, uint64_t n, int dtype, uint64_t max_total, Workspace* ws, uint64_t epoch,
                       HostResult* host, uint64_t (&met)[kMeetLines], int looks, hipStream_t s) {
    const u32 nchunks = (u32)num_chunks_of(n);
    OneDecArgs a = {blobs, w_ref, (u64)n, (u64)max_total, ws, host, (u64)epoch, {}, (u32)count, nchunks, 0, 0};
    // (one workgroup's chunk may take all that much longer than another's, with every blob)
    set_goals(a, nchunks, met, looks < 0 ? looks : looks * count);
#define LC_ONE(DT) do { if (count > 1) hipLaunchKernelGGL((k_decode_one<DT, true>), dim3(nchunks), dim3(kOneDecThreads), 0, s, a); \
                        else hipLaunchKernelGGL((k_decode_one<DT, false>), dim3(nchunks), dim3(kOneDecThreads), 0, s, a); } while (0)
    if (dtype == kF64) LC_ONE(kF64);
    else if (dtype == kBF16) LC_ONE(kBF16);
    else if (dtype == kF16) LC_ONE(kF16);
    else LC_ONE(kF32);
#undef LC_ONE
}

}  // namespace lc
