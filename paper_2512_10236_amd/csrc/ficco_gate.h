// Device side of a Gate (ficco_internal.h): how kernels wait for pieces. Not installed.
#pragma once
#include "ficco_internal.h"

namespace ficco {

// Bounded wait of one thread until a piece is ready (see Gate). Reads at system scope (past the
// caches): the writer is a copy engine. Returns 0 when the limit expires or another workgroup has
// already given up; the caller then skips its work, so every wave still reaches its exit.
static __device__ __forceinline__ int wait_ready(const Gate &g, int chunk)
{
    const uint64_t t0 = wall_clock64();
    const uint32_t *f = g.flags + (size_t)chunk * kFlagStrideWords;
    const int64_t *sv = g.sig_value ? reinterpret_cast<const int64_t *>(g.sig_value[chunk]) : nullptr;
    for (;;) {
        if (sv) {
            if (__hip_atomic_load(sv, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) <= 0) return 1;
        } else {
            if (__hip_atomic_load(f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) == g.epoch) return 1;
        }
        if (__hip_atomic_load(g.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) != 0u) return 0;
        if (wall_clock64() - t0 > g.spin_limit_ticks) {
            __hip_atomic_store(g.status, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            __hip_atomic_store(g.status_host, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            return 0;
        }
        __builtin_amdgcn_s_sleep(8);
    }
}

// One look at a piece, without waiting: has it landed?
static __device__ __forceinline__ int peek_ready(const Gate &g, int chunk)
{
    if (g.sig_value) return __hip_atomic_load(reinterpret_cast<const int64_t *>(g.sig_value[chunk]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) <= 0;
    return __hip_atomic_load(g.flags + (size_t)chunk * kFlagStrideWords, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) == g.epoch;
}

// The same for several pieces, piece_of(0) ... piece_of(n - 1), by one whole wavefront: lane l watches pieces l, l + 64,
// ... A look at a signal is a round trip to host memory of 1-2 us, and a wave that looked at its pieces one after the
// other paid one for each of them, landed or not; this way it pays one for 64. But hundreds of waves that look at all
// their pieces all the time swamp the host link, which the transfers' own signals cross too. So a wave looks at all of
// them first, then at the last one that is missing (pieces are listed in the order in which they leave), and at all again
// when that one has landed, every kLookEvery polls, and before it gives up; kLookFew pieces are few enough to be looked at
// all the time, which saves that last look. M 1675, K 3264, N 7496, eight experts in four steps, 32 pieces a tile: one after
// the other 590 us, all of them all the time 887-907, this way 579; M 2356, K 1280, N 7168, two experts, 4-5 pieces a tile 186,
// 202, 183 (193 with up to four at a time); one launch per step over eight shards, M 3072, K 5568, N 616, 202, 185, 169.
// The limit counts from the last time that a piece was seen to land. Returns the same value in every lane.
constexpr int kLookEvery = 8, kLookFew = 2;
template <class PieceFn>
static __device__ __forceinline__ int wait_ready_all(const Gate &g, int n, PieceFn piece_of)
{
    const int lane = threadIdx.x & 63;
    uint64_t t0 = wall_clock64();
    for (int base = 0; base < n; base += 64) {
        int waiting = base + lane < n;
        const int piece = piece_of(waiting ? base + lane : base);
        uint64_t missing = __ballot(waiting);
        int all = 1;
        for (int polls = 1;; ++polls) {
            const int landed = waiting && (all || lane == 63 - __builtin_clzll(missing)) && peek_ready(g, piece);
            if (landed) waiting = 0;
            missing = __ballot(waiting);
            if (!missing) {
                if (base + 64 < n) t0 = wall_clock64();      // the next 64 have the whole limit, as after any landing
                break;
            }
            const int any = __any(landed);
            if (any) t0 = wall_clock64();
            const int late = wall_clock64() - t0 > g.spin_limit_ticks;
            int give_up = 0;
            if (lane == 0) {
                if (__hip_atomic_load(g.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) != 0u) {
                    give_up = 1;
                } else if (late && all) {
                    __hip_atomic_store(g.status, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                    __hip_atomic_store(g.status_host, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                    give_up = 1;
                }
            }
            if (__any(give_up)) return 0;
            const int last_landed = any && !all;
            all = last_landed || late || polls % kLookEvery == 0 || __builtin_popcountll(missing) <= kLookFew;
            if (!last_landed) __builtin_amdgcn_s_sleep(8);
        }
    }
    return 1;
}

}  // namespace ficco
