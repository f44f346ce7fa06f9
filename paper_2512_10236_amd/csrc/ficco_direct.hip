// GEMM of few output tiles straight from a row-major weight: C[M, N] = A[M, K] * W[K, N] in one launch, without the
// packed copy of the weight that the other GEMM kernels read. Same MFMA, same k order, same operand roles as theirs,
// hence the same bits.
//
// What bounds it: a product of a few rows is the weight's way through the chip, once. The kernel therefore cuts the
// output into many narrow tiles (16 FM rows x 64 columns, a whole 128-byte line of a weight row), so that many CUs pull
// at once, and keeps a ring of S - 1 stages of 128 k values (20-32 KiB each, over 100 KiB a CU) in flight, which
// covers the latency of memory. The weight's fragments need 8 consecutive k of one column, which a row-major tile does
// not hold next to each other: ds_read_b64_tr_b16 transposes on the way out of LDS (16 lanes read 4 rows x 16
// columns, lane i gets column i).
//
// With FM = 1 a stage of 20 KiB takes 0.19 us and M 64, K 4096, N 768 8.6 us: 46-50 bytes a cycle, which is what a CU draws
// from beyond its L2 however much is in flight (64 from L2). Packing the weight first takes 3.9 us and, with the gap to the
// second launch, 6-7 of a call. With the stage's reads behind its loads instead of in front of them 11.7 us. Neither fewer
// bytes a stage (16 x 32 tiles, twice the CUs, 9.7: half of a weight line is drawn as a whole one), nor reads a stage ahead
// in a second register buffer (11.1), nor wavefronts of their own for the loads (10.2), nor idle CUs that pull the XCD's
// lines into its L2 a few stages ahead (no change) made it faster.
#include "ficco_internal.h"
#include "ficco_mfma.h"

namespace ficco {
namespace {

typedef short i16x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) i16x4_t lds_i16x4_t;

// A stage is two halves of 64 k values, a half 16 FM rows of A (128 bytes each, k contiguous) and then 64 rows of W
// (128 bytes each, 64 columns). 16-byte slots are swizzled: slot s of row r of A lies at s ^ ((r >> 1) & 7), as in the
// other kernels; of W at s ^ w_swizzle(r), which spreads the rows 0-3 and 8-11 that 32 lanes of a transposing read
// touch, 32 bytes each, over all 64 banks.
template <int FM_, int S_>
struct DirectCfg {
    static constexpr int FM = FM_, S = S_;
    static constexpr int BM = 16 * FM, BN = 64, BK = 128;
    static constexpr int A_HALF = BM * 128, W_HALF = 64 * 128, HALF = A_HALF + W_HALF, STAGE = 2 * HALF;
    static constexpr int LDS_BYTES = S * STAGE;
    static constexpr int THREADS = 256;
    static constexpr int LOADS = FM + 4;               // load instructions per wavefront per stage: 4 FM KiB of A and 16 KiB of W
    // With 16 MFMAs a stage they go between its loads, which take 64 cycles each while all four wavefronts issue theirs: M 64,
    // K 4096, N 768 17.9 -> 15.5 us, M 900, K 2048, N 1024 10.4 -> 9.5. With 4 or 8 nothing is gained (8.6 : 8.8, 11.6 : 11.4).
    static constexpr bool BETWEEN = FM == 4;
    static_assert(FM == 1 || FM == 2 || FM == 4, "whole blocks of A per wavefront");
    static_assert(S >= 3 && (S - 2) * LOADS < 64, "vmcnt has 6 bits");
    static_assert(LDS_BYTES <= 160 * 1024 - 64, "ring must fit one CU");
};

static __device__ __forceinline__ int w_swizzle(int row) { return 2 * (((row >> 1) & 1) | (((row >> 3) & 1) << 1)); }

template <class T>
__global__ __launch_bounds__(T::THREADS) void gemm_direct_kernel(DirectLaunch a)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = scalar(threadIdx.x >> 6);
    // tiles in 8 runs, one per XCD, rows fastest: the row tiles that read the same columns of W share an L2
    const int total = a.tiles_m * a.tiles_n, q8 = total >> 3, r8 = total & 7, xcd = blockIdx.x & 7;
    const int lid = (xcd < r8 ? xcd * (q8 + 1) : r8 * (q8 + 1) + (xcd - r8) * q8) + (blockIdx.x >> 3);
    const int row0 = lid % a.tiles_m * T::BM, col0 = lid / a.tiles_m * T::BN;
    const int rows_valid = min(T::BM, a.M - row0), cols_valid = min(T::BN, a.N - col0);
    const int K = scalar(a.K);
    const int KS = (K + T::BK - 1) / T::BK;
    const bool half_tail = (K & 64) != 0;              // the last stage has one half only

    const uint16_t *const A = scalar_base(a.A + (int64_t)row0 * K);
    const uint16_t *const W = scalar_base(a.W + col0);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;

    // Loads, 1 KiB (8 rows of 128 bytes) each. A: block b = i * 4 + wave of the stage's 4 FM, blocks of half 0 first.
    // Rows past the last one read the last one (they are not stored).
    uint32_t off_a[T::FM];
    int half_a[T::FM];
#pragma unroll
    for (int i = 0; i < T::FM; ++i) {
        const int b = i * 4 + wave;
        const int row = b % (2 * T::FM) * 8 + lane / 8;
        half_a[i] = b / (2 * T::FM);
        off_a[i] = (uint32_t)(min(row, rows_valid - 1) * K + ((lane % 8) ^ ((row >> 1) & 7)) * 8) * 2u;
    }
    // W: rows i * 32 + wave * 8 ... + 7 of a half; slots past the last column read the last one
    const int w_slot = min((lane % 8) ^ w_swizzle(wave * 8 + lane / 8), cols_valid / 8 - 1);
    uint32_t off_w[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) off_w[i] = (uint32_t)((i * 32 + wave * 8 + lane / 8) * a.N + w_slot * 8) * 2u;

    auto issue = [&](int k, uint32_t stage, auto behind) __attribute__((always_inline)) {
        // k values from here to the second half (which is the first again where K ends with it; it is then not used)
        const int up = half_tail && k == KS - 1 ? 0 : 64;
        const uint16_t *const ak = A + (int64_t)k * T::BK, *const wk = W + (int64_t)k * T::BK * a.N;
        static_for<T::FM>([&](auto i_c) __attribute__((always_inline)) {
            constexpr int i = decltype(i_c)::value;
            const int b = i * 4 + wave;
            set_lds_target<0>(lds0 + stage + half_a[i] * T::HALF + b % (2 * T::FM) * 1024);
            asm volatile("s_nop 0" ::: "memory");
            load_to_lds_16(ak + (half_a[i] ? up : 0), off_a[i]);
            behind(i_c);
        });
        static_for<4>([&](auto i_c) __attribute__((always_inline)) {
            constexpr int i = decltype(i_c)::value, half = i / 2;
            set_lds_target<half * T::HALF + T::A_HALF + i % 2 * 4096>(lds0 + stage + wave * 1024);
            asm volatile("s_nop 0" ::: "memory");
            load_to_lds_16(wk + (half ? (int64_t)up * a.N : 0), off_w[i % 2]);
            behind(std::integral_constant<int, T::FM + i>{});
        });
    };

    // fragments of 32 k values (step kk of a half): lane = row (column) lane % 16, k values 8 (lane / 16) ... + 7
    const int g = lane >> 4, j = lane & 15;
    const uint32_t fa0 = (uint32_t)j * 128u, fw0 = (uint32_t)((8 * g + (j >> 2)) * 128 + (((2 * wave + ((j & 3) >> 1)) ^ w_swizzle(8 * g + (j >> 2))) * 16) + (j & 1) * 8);
    f32x4_t acc[T::FM];
#pragma unroll
    for (int i = 0; i < T::FM; ++i) acc[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    // A stage's fragments into registers, and their products; between the two go the next loads, whose issue (16 cycles
    // each on an address path that the four wavefronts share) covers the reads' latency
    bf16x8_t fn[4], fm[4][T::FM];
    auto read = [&](uint32_t stage) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t base = stage + q / 2 * T::HALF, w = lds0 + base + T::A_HALF + q % 2 * 32 * 128 + fw0;
            union { i16x4_t h[2]; bf16x8_t v; } n;
            n.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_t *)(uintptr_t)w);
            n.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_t *)(uintptr_t)(w + 4 * 128));
            fn[q] = n.v;
#pragma unroll
            for (int i = 0; i < T::FM; ++i)
                fm[q][i] = *reinterpret_cast<const bf16x8_t *>(smem + base + fa0 + i * 16 * 128 + (((4 * (q % 2) + g) ^ ((j >> 1) & 7)) << 4));
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    constexpr int NMF = 4 * T::FM;         // MFMAs of a stage
    auto product = [&](auto m_c) __attribute__((always_inline)) {
        constexpr int q = decltype(m_c)::value / T::FM, i = decltype(m_c)::value % T::FM;
        acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fn[q], fm[q][i], acc[i], 0, 0, 0);
    };
    auto multiply = [&](bool whole) __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
        static_for<NMF / 2>([&](auto m) __attribute__((always_inline)) { product(m); });
        if (whole) static_for<NMF / 2>([&](auto m) __attribute__((always_inline)) { product(std::integral_constant<int, NMF / 2 + m.value>{}); });
    };
    // Behind load l of a stage's, where products go between the loads: products [l - 1, l) / (LOADS - 1) of them all.
    auto products_behind = [&](auto l_c) __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
        static_for<NMF>([&](auto m) __attribute__((always_inline)) {
            if constexpr (decltype(l_c)::value == 1 + m.value * (T::LOADS - 1) / NMF) product(m);
        });
        __builtin_amdgcn_sched_barrier(0);
    };
    const auto nothing = [](auto) {};
    // One barrier per stage: behind it stage k has landed for everyone, and everyone has read stage k - 1, whose place
    // the next loads take.
    auto meet = [&](auto in_flight) __attribute__((always_inline)) {
        wait_vmem<decltype(in_flight)::value>();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        wg_barrier();
    };

    const int ahead = min(KS, T::S - 1);
    for (int k = 0; k < ahead; ++k) issue(k, k * T::STAGE, nothing);
    uint32_t cur = 0, next = (T::S - 1) * T::STAGE;    // places in the ring of stage k and of stage k + S - 1
    int k = 0;
    for (; k + T::S - 1 < KS; ++k) {
        meet(std::integral_constant<int, (T::S - 2) * T::LOADS>{});
        read(cur);
        if constexpr (T::BETWEEN) {
            issue(k + T::S - 1, next, products_behind);
        } else {
            issue(k + T::S - 1, next, nothing);
            multiply(true);
        }
        cur = cur == (T::S - 1) * T::STAGE ? 0 : cur + T::STAGE;
        next = next == (T::S - 1) * T::STAGE ? 0 : next + T::STAGE;
    }
    static_for<T::S - 1>([&](auto t) __attribute__((always_inline)) {
        constexpr int left = T::S - 1 - decltype(t)::value;          // stages that are still to be multiplied
        if (left <= ahead) {
            meet(std::integral_constant<int, (left - 1) * T::LOADS>{});
            read(cur);
            multiply(!(half_tail && k == KS - 1));
            ++k;
            cur = cur == (T::S - 1) * T::STAGE ? 0 : cur + T::STAGE;
        }
    });

    // acc[i][v] is C[16 i + lane % 16][16 wave + 4 (lane / 16) + v]; N and with it cols_valid are multiples of 8
    const int n = 16 * wave + 4 * g;
#pragma unroll
    for (int i = 0; i < T::FM; ++i) {
        const int m = 16 * i + j;
        if (m < rows_valid && n < cols_valid)
            *reinterpret_cast<u32x2_t *>(a.C + (int64_t)(row0 + m) * a.N + col0 + n) =
                u32x2_t{pack2_bf16_rne(acc[i][0], acc[i][1]), pack2_bf16_rne(acc[i][2], acc[i][3])};
    }
}

typedef DirectCfg<1, 7> D16;
typedef DirectCfg<2, 6> D32;
typedef DirectCfg<4, 4> D64;

template <class T>
hipError_t launch_direct_t(const DirectLaunch &a, hipStream_t s)
{
    static hipError_t once = hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_direct_kernel<T>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS_BYTES);
    if (once != hipSuccess) return once;
    DirectLaunch b = a;
    b.tiles_m = (a.M + T::BM - 1) / T::BM;
    b.tiles_n = (a.N + T::BN - 1) / T::BN;
    hipLaunchKernelGGL(gemm_direct_kernel<T>, dim3((unsigned)(b.tiles_m * b.tiles_n)), dim3(T::THREADS), T::LDS_BYTES, s, b);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_direct(int row_blocks, const DirectLaunch &a, hipStream_t s)
{
    if (a.M < 1 || a.N < 8 || a.N % 8 || a.K < kBK || a.K % kBK || a.K > kMaxK || (int64_t)a.K * a.N * 2 > 0x7FFFFFFF) return hipErrorInvalidValue;
    switch (row_blocks) {
    case 1: return launch_direct_t<D16>(a, s);
    case 2: return launch_direct_t<D32>(a, s);
    case 4: return launch_direct_t<D64>(a, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace ficco
