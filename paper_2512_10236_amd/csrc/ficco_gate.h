// Device side of a Gate (ficco_internal.h): how kernels wait for pieces. Not installed.
#pragma once
#include "ficco_internal.h"

namespace ficco {

// The gate at byte `offset` of the kernel's arguments, loaded where it is used: kept in registers from tile to tile it would
// cost the k loops theirs (scalar registers spilled, and read back in every turn).
static __device__ __forceinline__ Gate gate_argument(size_t offset)
{
    typedef __attribute__((address_space(4))) const char *args_t;
    args_t args = (args_t)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(args));
    Gate g;
    g.flags = *(uint32_t * __attribute__((address_space(4))) const *)(args + offset + offsetof(Gate, flags));
    g.sig_value = *(const uint64_t * __attribute__((address_space(4))) const *)(args + offset + offsetof(Gate, sig_value));
    g.epoch = *(__attribute__((address_space(4))) const uint32_t *)(args + offset + offsetof(Gate, epoch));
    g.status = *(uint32_t * __attribute__((address_space(4))) const *)(args + offset + offsetof(Gate, status));
    g.status_host = *(uint32_t * __attribute__((address_space(4))) const *)(args + offset + offsetof(Gate, status_host));
    g.spin_limit_ticks = *(__attribute__((address_space(4))) const uint64_t *)(args + offset + offsetof(Gate, spin_limit_ticks));
    return g;
}

// Every load of a wait is over, also by the compiler's book (its other way is a wait in each turn of the k loop that follows).
static __device__ __forceinline__ void loads_done() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// Between two polls, about 0.1 us for each nap.
static __device__ __forceinline__ void nap(Pace pace)
{
    for (uint32_t i = 0; i < pace.naps; ++i) __builtin_amdgcn_s_sleep(4);
}

// Bounded wait of one thread until a piece is ready (see Gate); `pace`: pace_of(). Reads at system scope (past the
// caches): the writer is a copy engine. Returns 0 when the limit expires or another workgroup has
// already given up; the caller then skips its work, so every wave still reaches its exit.
static __device__ __forceinline__ int wait_ready(const Gate &g, int chunk, Pace pace)
{
    const uint64_t t0 = wall_clock64();
    uint32_t *f = g.flags + (size_t)chunk * kFlagStrideWords;
    const int64_t *sv = g.sig_value ? reinterpret_cast<const int64_t *>(g.sig_value[chunk]) : nullptr;
    int late = 0;
    for (uint32_t polls = poll_phase(blockIdx.x, pace.every);; ++polls) {
        if ((!sv || pace.every > 1) && __hip_atomic_load(f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) == g.epoch) return 1;
        if (late || polls % pace.every == 0) {
            if (sv && __hip_atomic_load(sv, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) <= 0) {
                if (pace.every > 1) __hip_atomic_store(f, g.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                return 1;
            }
            if (__hip_atomic_load(g.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) != 0u) return 0;
            if (late) {                    // that look was the last one
                __hip_atomic_store(g.status, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                __hip_atomic_store(g.status_host, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                return 0;
            }
        }
        late = wall_clock64() - t0 > g.spin_limit_ticks;
        nap(pace);
    }
}

// One look at a piece, without waiting: has it landed? passed_on: at its flag too; at_signal: at its signal.
static __device__ __forceinline__ int peek_ready(const Gate &g, int chunk, int passed_on, int at_signal)
{
    uint32_t *const f = g.flags + (size_t)chunk * kFlagStrideWords;
    if (!g.sig_value) return __hip_atomic_load(f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) == g.epoch;
    if (passed_on && __hip_atomic_load(f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) == g.epoch) return 1;
    if (!at_signal || __hip_atomic_load(reinterpret_cast<const int64_t *>(g.sig_value[chunk]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) > 0) return 0;
    if (passed_on) __hip_atomic_store(f, g.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    return 1;
}

// The same for several pieces, piece_of(0) ... piece_of(n - 1), by one whole wavefront: lane l watches pieces l, l + 64,
// ... A look at a signal is a round trip to host memory of 1-2 us, and a wave that looked at its pieces one after the
// other paid one for each of them, landed or not; this way it pays one for 64. But waves that look at all their pieces all
// the time swamp the host link, which the transfers' own signals cross too: PollPlan. M 1675, K 3264, N 7496, eight experts
// in four steps, 32 pieces a tile, every workgroup at the signals on every poll: one after the other 590 us, all of them all
// the time 887-907, this way 579.
// The limit counts from the last time that a piece was seen to land. Returns the same value in every lane.
template <class PieceFn>
static __device__ __forceinline__ int wait_ready_all(const Gate &g, int n, Pace pace, PieceFn piece_of)
{
    const int lane = threadIdx.x & 63;
    uint64_t t0 = wall_clock64();
    for (int base = 0; base < n; base += 64) {
        int waiting = base + lane < n;
        const int piece = piece_of(waiting ? base + lane : base);
        uint64_t missing = __ballot(waiting);
        int late = 0;
        for (PollPlan poll(pace.every, poll_phase(blockIdx.x, pace.every));;) {
            const int last = lane == 63 - __builtin_clzll(missing);
            const int landed = waiting && (poll.flags || last) &&
                               peek_ready(g, piece, pace.every > 1, (uint32_t)__builtin_popcountll(missing >> lane) <= poll.signals);
            const int last_landed = __any(landed && last);
            if (landed) waiting = 0;
            missing = __ballot(waiting);
            if (!missing) {
                if (base + 64 < n) t0 = wall_clock64();      // the next 64 have the whole limit, as after any landing
                break;
            }
            const int any = __any(landed);
            if (any) t0 = wall_clock64();
            const int last_look = late && !any;
            late = wall_clock64() - t0 > g.spin_limit_ticks;
            int give_up = 0;
            if (lane == 0 && poll.signals) {
                if (__hip_atomic_load(g.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) != 0u) {
                    give_up = 1;
                } else if (last_look) {
                    __hip_atomic_store(g.status, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                    __hip_atomic_store(g.status_host, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                    give_up = 1;
                }
            }
            if (__any(give_up)) return 0;
            poll.next(last_landed, late, (uint32_t)__builtin_popcountll(missing));
            if (!last_landed) nap(pace);
        }
    }
    loads_done();
    return 1;
}

}  // namespace ficco
