// Workgroups of one launch that wait for each other: k_encode_one and k_decode_one (gfx950).
#pragma once
#include "lc_device.h"

namespace lc {

// Everything that passes between workgroups goes through agent-scope atomic operations, whose completion each
// waits for before it arrives (no fence: writing back the L2 of a die from every workgroup costs more than the launches
// saved).  A workgroup may wait for one that has not started, because others' kernels hold the chip: the host launches
// this kernel only while all workgroups of such calls fit the chip together, and the wait is bounded.  It is given up by
// marking a counter that is not yet full, so either every counter filled up unmarked, and no one can give up any more, or one
// is marked, and no one finds them full; the first workgroup then does not report, and the host runs the call in several
// kernels.  A meeting of 64 workgroups takes 1.2 us, of 256 1.5 (one counter for all: 1.4 and 3.7).
struct GridMeeting {
    OneSync* sync;
    u64 goal;                // lane k: what counter k stands at when all have arrived
    u32 lines, limit;        // counters; how often to look
    // by one thread, behind the others' waits for their own operations; refuse: what the workgroups meet for is off
    __device__ __forceinline__ void arrive(u32 which, bool refuse = false) const {
        __hip_atomic_fetch_add(&sync->line[which][blockIdx.x % lines].arrived, refuse ? 1ull + kRefused : 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ unsigned long long* counter(u32 which) const { return &sync->line[which][lane_id() < lines ? lane_id() : 0].arrived; }
    __device__ __forceinline__ u64 look(u32 which) const { return __hip_atomic_load(counter(which), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    // By one wavefront: whether all have arrived and none refused.  seen: look(which), perhaps of some time ago.
    __device__ __forceinline__ bool wait(u32 which, u64 seen) const {
        const u32 lane = lane_id();
        for (u32 i = 0;; ++i) {
            if (__any(lane < lines && (seen & kGivenUp) != 0)) return false;
            const u64 missing = __ballot(lane < lines && (seen & (kRefused - 1)) != goal);
            if (missing == 0) return !__any(lane < lines && seen >= kRefused);
            if (i >= limit) {                        // (fails only if another has arrived there: at most as often as there are workgroups)
                bool marked = false;
                if (lane == (u32)__builtin_ctzll(missing))
                    marked = __hip_atomic_compare_exchange_strong(counter(which), &seen, seen | kGivenUp, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (__any(marked)) return false;
            } else if (i >= 64) __builtin_amdgcn_s_sleep(8);
            seen = look(which);
        }
    }
    __device__ __forceinline__ bool wait(u32 which) const { return wait(which, look(which)); }
};
// The host's side: the counters' goals for a grid of nchunks workgroups.  looks < 0: a goal that no arrival reaches, so that every
// workgroup gives up at its first look.
template <typename Args>
inline void set_goals(Args& a, uint32_t nchunks, uint64_t (&met)[kMeetLines], int looks) {
    a.lines = nchunks <= kMeetOneLine ? 1 : kMeetLines;
    a.limit = looks < 0 ? 0 : (u32)looks;
    for (u32 k = 0; k < a.lines; ++k) a.goal[k] = met[k] += (nchunks + a.lines - 1 - k) / a.lines;
    if (looks < 0) ++a.goal[0];
}
__device__ __forceinline__ void wait_own_operations() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
template <typename T> __device__ __forceinline__ T load_shared(const T* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

}  // namespace lc
