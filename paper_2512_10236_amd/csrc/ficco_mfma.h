// Device helpers the GEMM kernels share: vector types, the direct global -> LDS loads and their waits. Not installed.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>
#include <utility>

namespace ficco {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// two fp32 -> two bf16, round to nearest even, in one instruction (v_cvt_pk_bf16_f32)
static __device__ __forceinline__ uint32_t pack2_bf16_rne(float lo, float hi)
{
    const bf16x2_t v = {(__bf16)lo, (__bf16)hi};
    return __builtin_bit_cast(uint32_t, v);
}

template <int... I, class Fn>
static __device__ __forceinline__ void static_for_(std::integer_sequence<int, I...>, Fn &&f) { (f(std::integral_constant<int, I>{}), ...); }
// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>): a loop whose index is a constant in every turn
template <int N, class Fn>
static __device__ __forceinline__ void static_for(Fn &&f) { static_for_(std::make_integer_sequence<int, N>{}, f); }

// 64 lanes x 16 B from global memory straight into 1 KiB of LDS at the wave-uniform byte address in M0 (lane l lands
// at M0 + 16 l). The global address is a wave-uniform 64-bit base (scalar registers) plus a per-lane 32-bit byte
// offset, so that stepping along k costs scalar additions only and a load needs one vector register. Issued through
// inline assembly so that the waits are placed by hand (s_waitcnt vmcnt) and not widened by the compiler. M0 is
// written by an instruction of its own (set_lds_target), which the k loop places one MFMA ahead of the load: the wait
// state the hardware wants between the two is then an MFMA instead of a no-op, and no slot between two MFMAs has to
// take more than two instructions. Between a set_lds_target and its load there is no other use of M0 (the kernels
// use nothing that needs it: no GDS, no messages, no indirect registers).
//
// The base must be in scalar registers well before the load: a scalar register that a vector instruction has written
// (v_readfirstlane, which is what the compiler makes of an address it cannot prove uniform) may be read by a memory
// instruction only 5 wait states later, and the compiler, which sees to that for its own instructions, does not look
// into inline assembly. scalar_base() is the way in: it makes the two halves uniform, waits, and returns an opaque
// scalar, on which everything after it is scalar arithmetic. (tests/test_asm_hazards.py checks the assembly.)
static __device__ __forceinline__ const uint16_t *scalar_base(const uint16_t *p)
{
    const uint64_t b = (uint64_t)p;
    uint64_t s = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(b >> 32)) << 32) | (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)b);
    asm volatile("s_nop 4" : "+s"(s));
    return (const uint16_t *)s;
}
static __device__ __forceinline__ int scalar(int v) { return __builtin_amdgcn_readfirstlane(v); }
template <int IMM>
static __device__ __forceinline__ void set_lds_target(uint32_t lds_base)
{
    asm volatile("s_add_i32 m0, %0, %1" ::"s"(lds_base), "n"(IMM) : "m0", "scc");
}
static __device__ __forceinline__ void load_to_lds_16(const void *base, uint32_t lane_off)
{
    asm volatile("global_load_lds_dwordx4 %0, %1" ::"v"(lane_off), "s"(base) : "memory");
}
// 16 bytes per lane written through the caches (system scope), for data that a copy engine reads while the kernel runs on.
// The hardware reads the data of a store of more than 64 bits up to two wait states after its issue; the compiler keeps
// its vector instructions off the registers that long behind its own stores only, hence the no-op (without it up to 26
// stores of a tile's epilogue had their registers overwritten one state later; tests/test_asm_hazards.py checks it).
static __device__ __forceinline__ void store_through_16(void *dst, u32x4_t v)
{
    asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1\n\ts_nop 1" ::"v"(dst), "v"(v) : "memory");
}
template <int N>
static __device__ __forceinline__ void wait_vmem() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
static __device__ __forceinline__ void wg_barrier() { asm volatile("s_barrier" ::: "memory"); }

}  // namespace ficco
