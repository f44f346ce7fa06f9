// bf16 MFMA GEMM kernels for gfx950 (CDNA4): C[rows, N] = A[rows, K] * W[K, N], fp32 accumulate,
// one round-to-nearest-even to bf16 at the end.
//
// This is the "chunk GEMM" of the overlap path (paper Sec. II-B for the operation, Sec. V-A for
// launching it per landed piece or per step). Two entry kernels share one tile routine:
//   * gemm_blocks_kernel   - one launch over a list of equal-height row blocks (a monolithic GEMM,
//                            one landed piece, or the G pieces of a fused step read in place);
//   * gemm_resident_kernel - one launch for the whole run; workgroups draw tiles from a ticket
//                            counter in arrival order and wait until the tile's piece is ready.
//
// Data flow per workgroup tile (BM x BN, 256 threads = 4 wavefronts of 64):
//   global --global_load_lds_dwordx4--> LDS (a ring of stages of BK = 64, XOR-swizzled 16 B slots)
//   LDS --ds_read_b128--> 8-element bf16 fragments --> v_mfma_f32_16x16x32_bf16 --> fp32 accumulators
// The weight is read from a packed copy Wt[N, K] (k contiguous), so A and Wt fragments use the
// same access pattern. Every output element is accumulated over k ascending by the same
// instruction, whatever the tile shape or row block, which makes results bit-identical across
// schedules.
#include "ficco_internal.h"
#include "ficco_gate.h"
#include "ficco_mfma.h"
#include <stdlib.h>
#include <algorithm>

namespace ficco {

// A workgroup tile and the schedule of its k loop. The loop's unit is the slot: one v_mfma_f32_16x16x32_bf16 and what
// is issued behind it. A turn of TT slots multiplies one k-tile (a stage of 64 k values, two halves of 32); see
// tile_accumulate_from for what the positions mean.
template <int BM_, int BN_, int WGM_, int WGN_, int NSTAGE_>
struct TileCfg {
    static constexpr int BM = BM_, BN = BN_, WGM = WGM_, WGN = WGN_;
    static constexpr int NSTAGE = NSTAGE_;                     // LDS stages in the ring: the loads of k-tile k + NSTAGE follow the reads of k-tile k
    static constexpr int BK = kBK;
    static constexpr int ROWB = BK * 2;                        // bytes of a row of a stage
    static constexpr int SLOTS = BK / 8;                       // 16-byte slots per row
    static constexpr int RPL = 1024 / ROWB;                    // rows one load instruction (64 lanes x 16 B) fills
    static constexpr int THREADS = WGM * WGN * 64;
    static constexpr int WTM = BM / WGM, WTN = BN / WGN;       // wavefront tile
    static constexpr int FM = WTM / 16, FN = WTN / 16;         // 16x16 MFMA blocks per wavefront
    static constexpr int A_STAGE = BM * ROWB, B_STAGE = BN * ROWB;   // bytes
    static constexpr int STAGE = A_STAGE + B_STAGE;
    static constexpr int LDS_BYTES = NSTAGE * STAGE;
    static constexpr int NW = WGM * WGN;                       // wavefronts, one per SIMD
    static constexpr int AB = BM / RPL / NW, BB = BN / RPL / NW; // 1 KiB blocks loaded per wavefront per stage
    static constexpr int LOADS = AB + BB;                      // load instructions per wavefront per k-tile
    static constexpr int NM = FM * FN, TT = 2 * NM;            // MFMAs per half and per turn
    static constexpr int NR = FM + FN;                         // fragment reads per half
    // LDS hands a wavefront one 1 KiB fragment in about 32 cycles when all four read: a read every second slot where the
    // turn has the slots for it.
    static constexpr int RSTEP = TT >= 4 * NR ? 2 : 1;
    // Two stages: the stage is free (FREE) long before the other one is needed (LAND). More stages: one barrier does both.
    static constexpr bool SPLIT = NSTAGE == 2 && TT >= 64;
    static constexpr int R1 = SPLIT ? 6 : 0;                   // first slot of the reads of this k-tile's second half
    static constexpr int FREE = R1 + NR * RSTEP + (SPLIT ? 2 : RSTEP == 2 ? 4 : 3);
    static constexpr int LAND = SPLIT ? TT + 4 - 2 * (NR - 1) - 2 : FREE;
    static constexpr int R0 = SPLIT ? LAND + 2 : LAND + 1;     // first slot of the reads of the next k-tile's first half
    static constexpr int LS = FREE + 1;                        // first load of k-tile k + NSTAGE
    static constexpr int LSTEP = NSTAGE == 2 && !SPLIT ? 2 : TT / LOADS > 0 ? TT / LOADS : 1;
    static constexpr bool at(int dist, int step, int count) { return dist >= 0 && dist % step == 0 && dist / step < count; }
    static constexpr int load_slot(int l) { return LS + l * LSTEP; }
    static constexpr int loads_before(int slot) { int n = 0; for (int l = 0; l < LOADS; ++l) n += load_slot(l) < slot; return n; }
    static constexpr int WRAPPED = LOADS - loads_before(TT);   // loads that fall into the next turn
    // loads in flight at LAND that are younger than those of the next k-tile
    static constexpr int younger_at_land() { int n = 0; for (int e = 0; e + 2 <= NSTAGE; ++e) n += loads_before(LAND + e * TT); return n; }
    // First and last slot of a half whose MFMA uses fragment q (row block 0, the column blocks, the other row blocks; column
    // blocks go back and forth from row block to row block).
    static constexpr int first_use(int q) { return q == 0 ? 0 : q <= FN ? q - 1 : (q - FN) * FN; }
    static constexpr int last_use(int q)
    {
        return q == 0 ? FN - 1 : q <= FN ? (FM - 1) * FN + (FM % 2 ? q - 1 : FN - q) : (q - FN) * FN + FN - 1;
    }
    // A half's fragments are replaced behind their last MFMA and there before their first. (256x128 and 128x256 begin to
    // read the next k-tile's first half three MFMAs before this one's is done with.)
    static constexpr bool fragments_hold()
    {
        for (int q = 0; q < NR; ++q) {
            const int r0 = R0 + q * RSTEP, r1 = R1 + q * RSTEP;
            if (r0 < last_use(q) || (r0 >= TT && r0 - TT >= first_use(q)) || r1 >= NM + first_use(q)) return false;
        }
        return true;
    }
    // Stages go in pairs (tile_accumulate_burst).
    static constexpr bool BURST = NM <= 4;
    static_assert(BURST || fragments_hold(), "a fragment is read too early or too late");
    static_assert(BURST ? NSTAGE % 2 == 0 && NSTAGE >= 6 && (NSTAGE - 2) * LOADS < 64 : NSTAGE >= 2 && NSTAGE <= 6 && (NSTAGE - 1) * LOADS < 64,
                  "ring of 2 to 6 stages, or pairs of them, vmcnt has 6 bits");
    static_assert(LDS_BYTES <= 160 * 1024 - 64, "LDS ring plus the kernels' few static words must fit one CU");
    static_assert(THREADS == 256, "4 wavefronts");
    static_assert(BM % (RPL * NW) == 0 && BN % (RPL * NW) == 0, "every wavefront loads the same number of blocks");
    static_assert(WTM % 16 == 0 && WTN % 32 == 0, "wavefront tile is made of 16x16 blocks, stored in pairs along a row");
    static_assert(AB >= 1 && BB >= 1, "tile too small for the loader");
    static_assert(BURST || (R0 + (NR - 1) * RSTEP - TT < (FM - 1) * FN && R0 + (NR - 1) * RSTEP - TT < FREE && load_slot(LOADS - 1) - TT < LS && load_slot(LOADS - 1) < LAND + (NSTAGE - 1) * TT),
                  "what a turn leaves to the next one is done before it is needed");
};

// Computes one BM x BN tile. a_tile: first row of the tile in A; rows_valid in [1, BM] rows of
// it exist (the others are neither stored nor allowed to fault: their loads are clamped to the
// last valid row). wt_tile: first row (= output column) of the tile in Wt; cols_valid likewise.
//
// LDS holds a ring of NSTAGE stages; a stage is BM + BN rows of 128 B (64 k values), the 16-byte
// slot kc of row r stored at slot kc ^ ((r >> 1) & 7) so that the 16 lanes of a ds_read_b128 phase
// hit 64 different banks. Loads go global -> LDS directly (no staging registers): a wavefront
// instruction fills 8 rows, lane l fetching the slot that belongs at position l. The big tile only
// has room for two stages; the smaller tiles use three or four, which is what keeps launches with
// few workgroups (small pieces) from being bound by load latency. The loop itself is described in
// tile_accumulate_from.
template <class T>
struct TileAcc {
    f32x4_t acc[T::FN][T::FM];
};

template <class T>
static __device__ __forceinline__ void tile_zero(TileAcc<T> &ta)
{
#pragma unroll
    for (int j = 0; j < T::FN; ++j)
#pragma unroll
        for (int i = 0; i < T::FM; ++i) ta.acc[j][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    // the MFMAs are inline assembly, so the compiler does not know what they need after a write to their accumulators
    asm volatile("s_nop 7" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

struct NoHook {
    __device__ __forceinline__ void operator()() const {}
};

// Byte offset, from the first row of the tile, of what lane `lane` fetches for 1 KiB block `blk` of a stage:
// row blk*RPL + lane/SLOTS (clamped to the last row that exists), 16-byte slot (lane%SLOTS) ^ swizzle(row) of
// its k-tile. The swizzle - (row>>1)&7, two rows of 128 B share a 256-byte line of banks - spreads the rows over
// different slots, so that the 16 lanes of a ds_read_b128 phase, which read one k slot of 16 consecutive rows, hit 64
// different banks.
template <class T>
static __device__ __forceinline__ uint32_t lane_offset(int blk, int lane, int rows_valid, int64_t row_stride_elems)
{
    const int row = blk * T::RPL + lane / T::SLOTS;
    const int kc = (lane % T::SLOTS) ^ ((row >> 1) & (T::SLOTS - 1));
    const int rr = row < rows_valid ? row : rows_valid - 1;
    return (uint32_t)(((int64_t)rr * row_stride_elems + kc * 8) * 2);
}

// Where the loader finds its part of k-tile kt of A. PlainA: one row-major block [rows, K] with row stride lda:
// a wave-uniform base that moves along k, and one per-lane byte offset per load (the tile's rows must span less
// than 4 GiB, which the shape rules guarantee: at most 256 rows of at most 2^31 elements... of 2 bytes - the
// launchers refuse row strides above kMaxK).
template <class T>
struct PlainA {
    uint32_t off[T::AB];
    const uint16_t *base;
    __device__ __forceinline__ PlainA(const uint16_t *a_tile, int rows_valid, int64_t lda, int wave, int lane) : base(scalar_base(a_tile))
    {
#pragma unroll
        for (int i = 0; i < T::AB; ++i) off[i] = lane_offset<T>(wave * T::AB + i, lane, rows_valid, lda);
    }
    __device__ __forceinline__ void seek(int) {}
    __device__ __forceinline__ const uint16_t *at(int kt) const { return base + (int64_t)kt * T::BK; }
};

// SlicedA: a run of consecutive k slices of the K-sliced layout (slice s = the [M][k0[s+1]-k0[s]] block that
// starts at element M*k0[s]), read as one k range. The issue stream walks the k-tiles in ascending order;
// `seek` moves to the slice a k-tile lies in and only then rebuilds the base and the per-lane offsets for that
// slice's row stride, so that inside a slice a load costs what it costs with PlainA.
template <class T>
struct SlicedA {
    uint32_t off[T::AB];
    const uint16_t *base;
    const uint16_t *A;
    const int32_t *k0;
    int64_t M, row0;
    int sl, kt_begin, kt_end, rows_valid, wave, lane;
    __device__ __forceinline__ SlicedA(const uint16_t *A_, const int32_t *k0_, int64_t M_, int64_t row0_, int first_slice, int rows_valid_,
                                       int wave_, int lane_)
        : base(A_), A(A_), k0(k0_), M(M_), row0(row0_), sl(first_slice - 1), kt_begin(0), kt_end(0), rows_valid(rows_valid_), wave(wave_), lane(lane_)
    {
    }
    __device__ __forceinline__ void seek(int kt)
    {
        while (kt >= kt_end) {               // uniform: every lane takes the same steps
            ++sl;
            const int kb = scalar(k0[sl]), kw = scalar(k0[sl + 1]) - kb;
            kt_begin = kt_end;
            kt_end += kw / T::BK;
            base = scalar_base(A + M * kb + row0 * kw);
#pragma unroll
            for (int i = 0; i < T::AB; ++i) off[i] = lane_offset<T>(wave * T::AB + i, lane, rows_valid, kw);
        }
    }
    __device__ __forceinline__ const uint16_t *at(int kt) const { return base + (int64_t)(kt - kt_begin) * T::BK; }
};

// One MFMA: 16 columns of the packed weight x 16 rows of A x 32 k. The operands are passed swapped (D[n][m]), so that
// a lane ends up with 4 consecutive columns of one C row. Inline assembly with the accumulator tied to the
// accumulation registers: the builtin leaves the register allocator free to move the 256 of the big tile between the
// two halves of the register file, which it does with hundreds of copies per turn.
static __device__ __forceinline__ void mfma_16x16x32(f32x4_t &c, const bf16x8_t &n, const bf16x8_t &m)
{
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(n), "v"(m));
}

// The k loop of tiles whose turn has too few MFMAs to put anything behind. A turn is two stages (128 k values): one wait and
// one barrier, behind which its k-tiles have landed for everyone and everyone has read the two before; then all of its
// fragments out of LDS; then the loads that refill the two stages before it, with the MFMAs between them, as their fragments
// arrive (a wavefront's loads take 64 cycles each while all four issue theirs, and what is behind a load waits for that).
//
// What bounds it: the CU draws 64 bytes a cycle from L2 and 45-52 from beyond, whatever is in flight. 32x64 tiles draw 24 KiB
// a turn, 64x64 32 KiB, where 64x128 draws 48: 0.26 / 0.35 / 0.45 us, of which the loads alone are 0.22 / 0.31 / 0.45. MFMAs
// behind all loads 0.275 / 0.41; touching the lines a few turns ahead with a fifth wavefront 0.42 / 0.52, because a touched
// line takes the same way.
template <class T, class Hook, class AddrA>
static __device__ __forceinline__ void tile_accumulate_burst(TileAcc<T> &ta, AddrA &pa, const uint16_t *__restrict__ wt_tile, int cols_valid,
                                                             int64_t ldw, int K, unsigned char *smem, Hook after_first_wait)
{
    const int lane = threadIdx.x & 63;
    const int wave = scalar(threadIdx.x >> 6);
    const int wm = wave / T::WGN, wn = wave % T::WGN;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;
    const uint16_t *const wt = scalar_base(wt_tile);
    constexpr int TURNS = T::NSTAGE / 2, PAIR = 2 * T::STAGE, LOADS = 2 * T::LOADS;
    const int KT = scalar(K) / T::BK, KP = (KT + 1) / 2;
    uint32_t offb[T::BB];
#pragma unroll
    for (int i = 0; i < T::BB; ++i) offb[i] = lane_offset<T>(wave * T::BB + i, lane, cols_valid, ldw);
    // load l of a turn's: those of its first k-tile, then those of its second (which may not exist at the end of K: the first
    // again, and not used)
    auto load = [&](int t, uint32_t pair, auto l_c) __attribute__((always_inline)) {
        constexpr int u = decltype(l_c)::value / T::LOADS, l = decltype(l_c)::value % T::LOADS;
        const int kt = min(2 * t + u, KT - 1);
        if constexpr (l == 0) pa.seek(kt);
        if constexpr (l < T::AB) set_lds_target<u * T::STAGE + l * 1024>(lds0 + pair + wave * T::AB * 1024);
        else set_lds_target<u * T::STAGE + T::A_STAGE + (l - T::AB) * 1024>(lds0 + pair + wave * T::BB * 1024);
        asm volatile("s_nop 0" ::: "memory");
        if constexpr (l < T::AB) load_to_lds_16(pa.at(kt), pa.off[l]);
        else load_to_lds_16(wt + (int64_t)kt * T::BK, offb[l - T::AB]);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto issue = [&](int t, uint32_t pair) __attribute__((always_inline)) {
        static_for<LOADS>([&](auto l) __attribute__((always_inline)) { load(t, pair, l); });
    };
    const int frow = lane & 15, fh = lane >> 4, fs = (frow >> 1) & 7;
    const int a_base = (wm * T::WTM + frow) * T::ROWB, b_base = T::A_STAGE + (wn * T::WTN + frow) * T::ROWB;
    bf16x8_t fa[4][T::FM], fb[4][T::FN];
    auto read = [&](uint32_t pair) __attribute__((always_inline)) {
        static_for<4>([&](auto h_c) __attribute__((always_inline)) {
            constexpr int h = decltype(h_c)::value;
            const unsigned char *base = smem + pair + h / 2 * T::STAGE + (((4 * (h % 2) + fh) ^ fs) << 4);
#pragma unroll
            for (int i = 0; i < T::FM; ++i) fa[h][i] = *reinterpret_cast<const bf16x8_t *>(base + a_base + i * 16 * T::ROWB);
#pragma unroll
            for (int j = 0; j < T::FN; ++j) fb[h][j] = *reinterpret_cast<const bf16x8_t *>(base + b_base + j * 16 * T::ROWB);
        });
        __builtin_amdgcn_sched_barrier(0);
    };
    constexpr int NMF = 4 * T::NM;         // MFMAs of a turn
    auto product = [&](auto m_c) __attribute__((always_inline)) {
        constexpr int m = decltype(m_c)::value, h = m / T::NM, i = m % T::NM / T::FN, j = m % T::FN;
        mfma_16x16x32(ta.acc[j][i], fb[h][j], fa[h][i]);
    };
    auto meet = [&](auto in_flight) __attribute__((always_inline)) {
        wait_vmem<decltype(in_flight)::value>();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        wg_barrier();
    };
    const int ahead = min(KP, TURNS - 1);
    for (int t = 0; t < ahead; ++t) issue(t, t * PAIR);
    uint32_t cur = 0, next = (TURNS - 1) * PAIR;
    int k = 0;
#pragma clang loop unroll(disable)
    for (; k + TURNS - 1 < KP; ++k) {
        meet(std::integral_constant<int, (TURNS - 2) * LOADS>{});
        if (k == 0) after_first_wait();
        read(cur);
        static_for<LOADS>([&](auto l) __attribute__((always_inline)) {
            load(k + TURNS - 1, next, l);
            static_for<NMF>([&](auto m) __attribute__((always_inline)) {
                if constexpr (l.value == 1 + m.value * (LOADS - 1) / NMF) product(m);
            });
            __builtin_amdgcn_sched_barrier(0);
        });
        cur = cur == (TURNS - 1) * PAIR ? 0 : cur + PAIR;
        next = next == (TURNS - 1) * PAIR ? 0 : next + PAIR;
    }
    static_for<TURNS - 1>([&](auto t) __attribute__((always_inline)) {
        constexpr int left = TURNS - 1 - decltype(t)::value;
        if (left <= ahead) {
            meet(std::integral_constant<int, (left - 1) * LOADS>{});
            if (k == 0) after_first_wait();
            read(cur);
            static_for<NMF / 2>([&](auto m) __attribute__((always_inline)) { product(m); });
            if (2 * k + 1 < KT) static_for<NMF / 2>([&](auto m) __attribute__((always_inline)) { product(std::integral_constant<int, NMF / 2 + m.value>{}); });
            ++k;
            cur = cur == (TURNS - 1) * PAIR ? 0 : cur + PAIR;
        }
    });
    // accumulators may be read after the last MFMA's passes
    asm volatile("s_nop 15" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// The k loop. Turn k multiplies k-tile k out of registers: slots [0, NM) its first half (k values 0..31 of the stage),
// whose fragments were read during the turn before, slots [NM, TT) its second half, whose fragments are read during
// the first (from slot R1 on). Behind the MFMAs go, at fixed slots (TileCfg),
//   FREE   all of this wavefront's reads of the stage are in registers; barrier: that holds for every wavefront
//   LS...  the loads of k-tile k + NSTAGE into the stage just freed, one every LSTEP slots, spread over a whole turn:
//          the last WRAPPED of them fall into turn k + 1
//   LAND   k-tile k + 1 has landed for this wavefront's loads; barrier: for everyone's
//   R0...  the reads of the first half of k-tile k + 1
// so that no wait ever has an MFMA's operands behind it, a load has between half a turn and a turn and a half (two
// stages) to arrive, and the address path, which takes 16 cycles per load and is shared by the four wavefronts, sees
// them evenly. All issue order is pinned (sched_barrier); what the compiler adds are the LDS waits of the fragments.
//
// What it measured on the 256x256 tile (M 4096, K 16384, N 4096: one round of tiles; random data, board at its 1400 W):
// v_mfma_f32_32x32x16 in this loop 1326 TFLOP/s, v_mfma_f32_16x16x32 1399 (half the accumulator traffic per flop, and
// the same bits); its loads spread over the turn instead of one every four slots 1512 (a denser issue holds up the
// MFMAs behind it); M0 written a slot ahead of its load 1552; this loop's row-segment stores 1556. The loop before it
// (32x32x16, one barrier per turn, the loads of a k-tile within half a turn) 1244; the vendor library 1596-1650.
// Counters (M 16384, K 8192, N 3584): 2446 cycles a turn, epilogues included, of which 2048 are MFMAs.
template <class T, class Hook = NoHook, class AddrA = PlainA<T>>
static __device__ __forceinline__ void tile_accumulate_from(TileAcc<T> &ta, AddrA &pa,
                                                            const uint16_t *__restrict__ wt_tile, int cols_valid,
                                                            int64_t ldw, int K, unsigned char *smem,
                                                            Hook after_first_wait = Hook())
{
    if constexpr (T::BURST) {
        tile_accumulate_burst<T, Hook, AddrA>(ta, pa, wt_tile, cols_valid, ldw, K, smem, after_first_wait);
        return;
    } else {
    f32x4_t (&acc)[T::FN][T::FM] = ta.acc;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / T::WGN, wn = wave % T::WGN;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;
    const uint16_t *const wt = scalar_base(wt_tile);
    constexpr int D = T::NSTAGE;           // k-tiles between a stage's reads and the loads that refill it

    uint32_t offb[T::BB];                  // per-lane byte offsets of the W loads from the tile's first row
#pragma unroll
    for (int i = 0; i < T::BB; ++i) offb[i] = lane_offset<T>(wave * T::BB + i, lane, cols_valid, ldw);
    // load l of the wavefront's LOADS loads of a k-tile: first the AB blocks of A, then the BB blocks of W (k-tiles are
    // issued in ascending order; load 0 of a k-tile comes first)
    const uint32_t lds_a = lds0 + wave * T::AB * 1024, lds_b = lds0 + T::A_STAGE + wave * T::BB * 1024;
    auto aim = [&](uint32_t stage, auto l_c) __attribute__((always_inline)) {
        constexpr int l = decltype(l_c)::value;
        if constexpr (l < T::AB) set_lds_target<l * 1024>(lds_a + stage);
        else set_lds_target<(l - T::AB) * 1024>(lds_b + stage);
    };
    auto load = [&](int kt, auto l_c) __attribute__((always_inline)) {
        constexpr int l = decltype(l_c)::value;
        if constexpr (l == 0) pa.seek(kt);
        if constexpr (l < T::AB) load_to_lds_16(pa.at(kt), pa.off[l]);
        else load_to_lds_16(wt + (int64_t)kt * T::BK, offb[l - T::AB]);
    };

    // LDS -> fragment addresses: lane reads row (lane%16) of a 16-row block, k-slot 4*half + lane/16,
    // un-swizzled by the row's swizzle, which only depends on the lane
    const int frow = lane & 15, fh = lane >> 4, fs = (frow >> 1) & 7;
    const int a_base = (wm * T::WTM + frow) * T::ROWB;
    const int b_base = T::A_STAGE + (wn * T::WTN + frow) * T::ROWB;
    bf16x8_t fa[2][T::FM], fb[2][T::FN];
    // fragment q of the FM + FN fragments of a half: the order of their first use (row block 0, every column block,
    // the other row blocks)
    auto read_frag = [&](uint32_t stage, auto half_c, auto q_c) __attribute__((always_inline)) {
        constexpr int half = decltype(half_c)::value, q = decltype(q_c)::value;
        const int slot = ((4 * half + fh) ^ fs) << 4;
        const unsigned char *base = smem + stage + slot;
        if constexpr (q == 0) fa[half][0] = *reinterpret_cast<const bf16x8_t *>(base + a_base);
        else if constexpr (q <= T::FN) fb[half][q - 1] = *reinterpret_cast<const bf16x8_t *>(base + b_base + (q - 1) * 16 * T::ROWB);
        else fa[half][q - T::FN] = *reinterpret_cast<const bf16x8_t *>(base + a_base + (q - T::FN) * 16 * T::ROWB);
    };
    constexpr std::integral_constant<int, 0> first{};
    constexpr std::integral_constant<int, 1> second{};

    // Past the last k-tile the loads go on, on the last k-tile again and into stages that are not read any more: every
    // turn is then the same code, which is what keeps the accumulators where they are (with a turn of its own for the
    // end of a tile the compiler copies all 256 of them between the two).
    const int KT = scalar(K) / T::BK;
    // ---- prologue: the loads of the first D k-tiles, except those that turn 0 issues itself
    static_for<D>([&](auto d) __attribute__((always_inline)) {
        static_for<T::LOADS>([&](auto l) __attribute__((always_inline)) {
            if constexpr (d.value < D - 1 || l.value < T::LOADS - T::WRAPPED) {
                aim(d.value * T::STAGE, l);
                asm volatile("s_nop 0" ::: "memory");
                load(min(d.value, KT - 1), l);
            }
        });
    });
    wait_vmem<(D - 1) * T::LOADS - T::WRAPPED>();
    wg_barrier();                          // k-tile 0 has landed for everyone
    after_first_wait();
    static_for<T::NR>([&](auto q) __attribute__((always_inline)) { read_frag(0, first, q); });

    if constexpr (T::at(T::TT - T::LS, T::LSTEP, T::LOADS)) aim((D - 1) * T::STAGE, std::integral_constant<int, (T::TT - T::LS) / T::LSTEP>{});
    uint32_t st_prev = (D - 1) * T::STAGE, st_cur = 0;         // byte offsets in the ring of the stages of k-tiles k - 1 and k
#pragma clang loop unroll(disable)
    for (int k = 0; k < KT; ++k) {
        const uint32_t st_next = st_cur == (D - 1) * T::STAGE ? 0 : st_cur + T::STAGE;
        const int kt = min(k + D, KT - 1), kt_wrapped = min(k + D - 1, KT - 1);
        static_for<T::TT>([&](auto p_c) __attribute__((always_inline)) {
            constexpr int p = decltype(p_c)::value;
            constexpr int half = p / T::NM, w = p % T::NM, i = w / T::FN;
            constexpr int j = i % 2 ? T::FN - 1 - w % T::FN : w % T::FN;       // back and forth: one operand stays from MFMA to MFMA
            mfma_16x16x32(acc[j][i], fb[half][j], fa[half][i]);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (T::at(p - T::R1, T::RSTEP, T::NR)) read_frag(st_cur, second, std::integral_constant<int, (p - T::R1) / T::RSTEP>{});
            if constexpr (p == T::FREE) {
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                if constexpr (T::FREE == T::LAND) wait_vmem<T::younger_at_land()>();
                wg_barrier();
            }
            if constexpr (p == T::LAND && T::FREE != T::LAND) {
                wait_vmem<T::younger_at_land()>();
                wg_barrier();
            }
            // a load, then the target of the next slot's
            if constexpr (T::at(p + T::TT - T::LS, T::LSTEP, T::LOADS)) load(kt_wrapped, std::integral_constant<int, (p + T::TT - T::LS) / T::LSTEP>{});
            if constexpr (T::at(p - T::LS, T::LSTEP, T::LOADS)) load(kt, std::integral_constant<int, (p - T::LS) / T::LSTEP>{});
            constexpr int n = (p + 1) % T::TT;
            if constexpr (T::at(n + T::TT - T::LS, T::LSTEP, T::LOADS))
                aim(p + 1 < T::TT ? st_prev : st_cur, std::integral_constant<int, (n + T::TT - T::LS) / T::LSTEP>{});
            if constexpr (T::at(n - T::LS, T::LSTEP, T::LOADS)) aim(st_cur, std::integral_constant<int, (n - T::LS) / T::LSTEP>{});
            // (in a tile's last turn these read a stage that is not used again)
            if constexpr (T::at(p - T::R0, T::RSTEP, T::NR)) read_frag(st_next, first, std::integral_constant<int, (p - T::R0) / T::RSTEP>{});
            if constexpr (T::at(p + T::TT - T::R0, T::RSTEP, T::NR)) read_frag(st_cur, first, std::integral_constant<int, (p + T::TT - T::R0) / T::RSTEP>{});
            __builtin_amdgcn_sched_barrier(0);
        });
        st_prev = st_cur;
        st_cur = st_next;
    }
    // accumulators may be read after the last MFMA's 16 passes
    asm volatile("s_nop 15\n\ts_nop 7" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    }
}

template <class T, class Hook = NoHook>
static __device__ __forceinline__ void tile_accumulate(TileAcc<T> &ta, const uint16_t *__restrict__ a_tile, int rows_valid,
                                                       const uint16_t *__restrict__ wt_tile, int cols_valid,
                                                       int64_t lda, int64_t ldw, int K, unsigned char *smem,
                                                       Hook after_first_wait = Hook())
{
    PlainA<T> pa(a_tile, rows_valid, lda, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), threadIdx.x & 63);
    tile_accumulate_from<T, Hook, PlainA<T>>(ta, pa, wt_tile, cols_valid, ldw, K, smem, after_first_wait);
}

// Rounds the accumulators to bf16 (nearest even) and stores the valid part of the tile.
// acc[j][i][v] is C[m][n] with m = wm*WTM + 16 i + lane%16, n = wn*WTN + 16 j + 4 (lane/16) + v. The lanes of odd rows
// of 16 exchange their half of column block j for their neighbours' half of block j + 1 (v_permlane16_swap), after
// which a lane holds 8 consecutive columns: a store instruction writes 16 bytes per lane, 64 bytes in each of 16 rows,
// and the two instructions of 64 columns whole lines. (8-byte stores without the exchange: twice the requests, and
// with the conversion done in integer arithmetic 6700 cycles more per 256x256 tile; M 65536, K 4096, N 14336: 5281 ->
// 5124 us.) THROUGH: written through the caches (system scope), for output that a copy engine reads while the kernel
// runs on. N and with it cols_valid are multiples of 8.
template <class T, bool THROUGH = false>
static __device__ __forceinline__ void tile_store(const TileAcc<T> &ta, uint16_t *__restrict__ c_tile, int rows_valid,
                                                  int cols_valid, int64_t ldc)
{
    const f32x4_t (&acc)[T::FN][T::FM] = ta.acc;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave / T::WGN, wn = wave % T::WGN;
    const int frow = lane & 15, fh = lane >> 4;
    const int n0 = wn * T::WTN + (fh & 1) * 16 + (fh >> 1) * 8;
#pragma unroll
    for (int i = 0; i < T::FM; ++i) {
        const int m = wm * T::WTM + i * 16 + frow;
        uint16_t *crow = c_tile + (int64_t)m * ldc;
#pragma unroll
        for (int j = 0; j < T::FN; j += 2) {
            const auto lo = __builtin_amdgcn_permlane16_swap(pack2_bf16_rne(acc[j][i][0], acc[j][i][1]),
                                                             pack2_bf16_rne(acc[j + 1][i][0], acc[j + 1][i][1]), false, false);
            const auto hi = __builtin_amdgcn_permlane16_swap(pack2_bf16_rne(acc[j][i][2], acc[j][i][3]),
                                                             pack2_bf16_rne(acc[j + 1][i][2], acc[j + 1][i][3]), false, false);
            const u32x4_t v = {lo[0], hi[0], lo[1], hi[1]};
            const int n = n0 + j * 16;
            if (m < rows_valid && n < cols_valid) {
                if constexpr (THROUGH) store_through_16(crow + n, v);
                else *reinterpret_cast<u32x4_t *>(crow + n) = v;
            }
        }
    }
}

template <class T>
static __device__ __forceinline__ void compute_tile(const uint16_t *__restrict__ a_tile, int rows_valid,
                                                    const uint16_t *__restrict__ wt_tile, int cols_valid,
                                                    uint16_t *__restrict__ c_tile, int64_t lda, int64_t ldw,
                                                    int64_t ldc, int K, unsigned char *smem)
{
    TileAcc<T> ta;
    tile_zero(ta);
    tile_accumulate<T>(ta, a_tile, rows_valid, wt_tile, cols_valid, lda, ldw, K, smem);
    tile_store<T>(ta, c_tile, rows_valid, cols_valid, ldc);
}

// Workgroups are dispatched round-robin over the 8 XCDs (each with its own L2). The tiles are cut
// into 8 runs of consecutive logical ids, one per XCD, and the tile grid is walked in groups of
// group_m row tiles, so that one XCD works on few A row tiles and W column tiles at a time. A launch
// with more tiles than the machine holds workgroups is started with that many workgroups only, and a
// workgroup takes every stride-th tile of its XCD's run: what is in flight on an XCD is the same run of
// ids that one workgroup per tile would give, without a workgroup start per tile.
struct XcdRun { int start, count, first, stride; };
static __device__ __forceinline__ XcdRun xcd_run(int pid, int grid, int total)
{
    const int q = total >> 3, r = total & 7;
    const int xcd = pid & 7;
    return {xcd < r ? xcd * (q + 1) : r * (q + 1) + (xcd - r) * q, q + (xcd < r ? 1 : 0), pid >> 3, (grid - xcd + 7) >> 3};
}

template <class T>
__global__ __launch_bounds__(T::THREADS) void gemm_blocks_kernel(GemmLaunch a)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    if (a.n_wait > 0) {
        __shared__ int s_go;
        if (threadIdx.x < 64) {
            const int ok = wait_ready_all(a.gate, a.n_wait, pace_of(gridDim.x, gridDim.x), [&](int i) { return a.wait_chunks[i]; });
            if (threadIdx.x == 0) s_go = ok;
        }
        __syncthreads();                   // also orders the tile's loads after the flag reads
        if (!s_go) return;
    }
    const int tiles_n = (a.N + T::BN - 1) / T::BN;
    const int rt_per_block = (a.rows_per_block + T::BM - 1) / T::BM;
    const int tiles_m = a.n_blocks * rt_per_block;
    const int total = tiles_m * tiles_n;
    const XcdRun run = xcd_run(blockIdx.x, gridDim.x, total);
    const int per_group = a.group_m * tiles_n;
    for (int t = run.first; t < run.count; t += run.stride) {
        const int lid = run.start + t;
        const int group = lid / per_group;
        const int first_m = group * a.group_m;
        const int gsz = min(tiles_m - first_m, a.group_m);
        const int tm = first_m + (lid % per_group) % gsz;
        const int tn = (lid % per_group) / gsz;

        const int blk = tm / rt_per_block, rt = tm % rt_per_block;
        const int brow0 = a.block_row0 ? a.block_row0[blk] : a.row0;
        const int64_t row0 = (int64_t)brow0 + (int64_t)rt * T::BM;
        const int rows_valid = min(T::BM, a.rows_per_block - rt * T::BM);
        const int col0 = tn * T::BN;
        const int cols_valid = min(T::BN, a.N - col0);
        compute_tile<T>(a.A + row0 * a.lda, rows_valid, a.Wt + (int64_t)col0 * a.K, cols_valid,
                        a.C + row0 * a.ldc + col0, a.lda, a.K, a.ldc, a.K, smem);
        __syncthreads();                   // everyone is done with the ring before the next tile refills it
    }
    wait_vmem<0>();                        // no load may arrive in LDS that is not this workgroup's any more
}

// Tile order of the resident kernels. Row tiles are numbered in arrival order (R = arrival position x
// row tiles per piece + row tile in the piece) and dealt round-robin to kTicketLists lists, one per
// XCD, each with its own ticket counter: a workgroup first serves the list of the XCD it presumably
// runs on (workgroups are dispatched round-robin over the XCDs), so that the tiles sharing an L2 at
// any time are few row tiles times a run of column tiles, and then helps the other lists. Inside a
// list tiles go in groups of a few row tiles, row tile fastest: as many as one step delivers to the
// list (so that no workgroup draws a tile of the next step while tiles of this one are left), 1 to 8.
// When a step delivers few row tiles and there are many column tiles, one row tile times all columns
// per XCD would stream the whole weight through every L2 once per round; the row-piece kernel then
// splits the lists by column block as well (ResidentLaunch::col_lists), so that an XCD works on
// several row tiles of the step times a run of columns, as a launch over the step's pieces would.
//
// TileWalk hands a workgroup its next (list, tile) pair. The first `rounds` tiles of its home list are the workgroup's
// by its rank among the workgroups that start there (no memory access), and short launches have all their tiles that way
// (hand_out); later tiles are drawn from the list's counter. Before it turns to the other lists it reads their counters once, all
// loads in flight together: on a list that is already used up it only leaves its one past-the-end draw (an atomic
// whose result nobody waits for), and a list that the ranks of its own workgroups cover completely is never drawn from
// at all. Counter traffic is what a launch pays at its end, since a draw goes to memory shared by all XCDs.
struct TileWalk {
    int turn;        // lists visited so far; the current list is (home + turn) % kTicketLists
    int taken;       // tiles of the home list taken by rank so far
    int looked;      // the other lists' counters have been read
    int spent;       // bit k: list (home + k) % kTicketLists was already used up at that look
    int x, t;        // the result: list and tile in the list, x < 0 when there is nothing left
    int have_drawn;  // `drawn` holds a counter value drawn ahead of time (kept here and not in a register across the k
    uint32_t drawn;  // loop, which leaves none: the compiler would spill it to memory)
};

// Issues, ahead of time, the draw that the next tile_walk_next() call would start with (if it would
// start with one) and returns 1 with the raw counter value in `drawn`; the caller puts this before
// work whose duration then hides the draw's round trip. Returns 0 when the next step is not a plain draw.
template <class TotalFn>
static __device__ __forceinline__ int tile_walk_predraw(const TileWalk &w, uint32_t *ticket, int grid, HandOut out, TotalFn total_of,
                                                        uint32_t &drawn)
{
    const int rounds = out.rounds;
    if (out.by_rank || w.turn >= kTicketLists || (w.turn == 0 && w.taken < rounds)) return 0;
    const int y = (blockIdx.x + w.turn) % kTicketLists;
    if (total_of(y) <= rounds * resident_list_homes(grid, y)) return 0;
    if (w.turn > 0 && (!w.looked || ((w.spent >> w.turn) & 1))) return 0;
    drawn = __hip_atomic_fetch_add(ticket + y * kFlagStrideWords, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return 1;
}

template <class TotalFn>
static __device__ __forceinline__ void tile_walk_next(TileWalk &w, uint32_t *ticket, const uint32_t *base, int grid, HandOut out,
                                                      TotalFn total_of)
{
    const int home = blockIdx.x % kTicketLists, rank = blockIdx.x / kTicketLists, rounds = out.rounds;
    w.x = -1;
    if (__builtin_expect(out.by_rank, 0)) {
        if (w.taken < rounds && !tile_by_rank(home, rank, w.taken, grid, rounds, total_of, w.x, w.t)) w.taken = rounds;
        ++w.taken;
        return;
    }
    while (w.turn < kTicketLists) {
        const int y = (home + w.turn) % kTicketLists;
        const int total = total_of(y), homes = resident_list_homes(grid, y);
        uint32_t *ctr = ticket + y * kFlagStrideWords;
        if (w.turn == 0 && w.taken < rounds) {
            const int cand = rank + w.taken * homes;
            ++w.taken;
            if (cand < total) { w.x = y; w.t = cand; return; }
            w.taken = rounds;                      // and none further on
        }
        if (total <= rounds * homes) {
            // the ranks of the workgroups that start on this list cover it: nobody draws from its counter
            ++w.turn;
            continue;
        }
        if (w.turn > 0 && !w.looked) {
            uint32_t seen[kTicketLists];
#pragma unroll
            for (int k = 1; k < kTicketLists; ++k)
                seen[k] = __hip_atomic_load(ticket + ((home + k) % kTicketLists) * kFlagStrideWords, __ATOMIC_RELAXED,
                                            __HIP_MEMORY_SCOPE_AGENT);
            int spent = 0;
#pragma unroll
            for (int k = 1; k < kTicketLists; ++k) {
                const int yk = (home + k) % kTicketLists;
                const int by_rank = rounds * resident_list_homes(grid, yk), total_k = total_of(yk);
                if (total_k > by_rank && (int)(seen[k] - base[yk]) + by_rank >= total_k) spent |= 1 << k;
            }
            w.spent = spent;
            w.looked = 1;
        }
        if (w.turn > 0 && ((w.spent >> w.turn) & 1)) {
            (void)__hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // result unused: no wait
            ++w.turn;
            continue;
        }
        const uint32_t raw = w.have_drawn ? w.drawn : __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        w.have_drawn = 0;
        const int cand = (int)(raw - base[y]) + rounds * homes;
        if (cand < total) { w.x = y; w.t = cand; return; }
        ++w.turn;                                  // that was this workgroup's one draw past the end of list y
    }
}

// The lists of a resident launch as a grid of row classes x column blocks (see resident_list_tiles):
// which tiles list x holds and where tile t of it lies. Inside a list tiles go in groups of `group`
// row tiles, row tile fastest.
struct ListGrid {
    int row_tiles, tiles_n, group;
    int cl_shift;                // log2 of the number of column blocks (1, 2, 4 or 8 of them): shifts, not divisions
    __device__ __forceinline__ ListGrid(int row_tiles_, int tiles_n_, int col_lists, int group_)
        : row_tiles(row_tiles_), tiles_n(tiles_n_), group(group_), cl_shift(31 - __clz(col_lists)) {}
    __device__ __forceinline__ int class_shift() const { return 3 - cl_shift; }              // kTicketLists = 8 lists
    __device__ __forceinline__ int row_class(int x) const { return x & ((1 << class_shift()) - 1); }
    __device__ __forceinline__ int col_block(int x) const { return x >> class_shift(); }
    __device__ __forceinline__ int rows(int x) const
    {
        const int rc = row_class(x);
        return row_tiles > rc ? (row_tiles - rc + (1 << class_shift()) - 1) >> class_shift() : 0;
    }
    __device__ __forceinline__ int col_begin(int x) const { return (col_block(x) * tiles_n) >> cl_shift; }
    __device__ __forceinline__ int cols(int x) const { return (((col_block(x) + 1) * tiles_n) >> cl_shift) - col_begin(x); }
    __device__ __forceinline__ int total(int x) const { return rows(x) * cols(x); }
    // tile t of list x: R = its row tile in the arrival-ordered sequence, tn = its column tile
    __device__ __forceinline__ void position(int x, int t, int &R, int &tn) const
    {
        const int my_rows = rows(x), my_cols = cols(x);
        const int per_group = group * my_cols;
        const int g = t / per_group, first = g * group;
        const int gsz = min(my_rows - first, group);
        R = ((first + (t % per_group) % gsz) << class_shift()) + row_class(x);
        tn = col_begin(x) + (t % per_group) / gsz;
    }
};
static_assert(kTicketLists == 8, "ListGrid shifts assume 8 lists");

// A workgroup of a resident kernel has read everything it will read of A when it gets here (the data went
// through the MFMAs before its last tile was stored), so the last one out may let the next run's transfers
// into A start.
__device__ __forceinline__ void leave_run(const RunExit &e)
{
    if (e.release_value && threadIdx.x == 0) {
        const uint32_t before = __hip_atomic_fetch_add(e.count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (before + 1u == e.target)
            __hip_atomic_store(e.release_value, (int64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// STREAM_OUT: the GEMM -> reduce-scatter form (r.done_count set), a separate instantiation so that its
// epilogue and bookkeeping cost the all-gather form no registers.
template <class T, bool STREAM_OUT>
__global__ __launch_bounds__(T::THREADS) void gemm_resident_kernel(ResidentLaunch r)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    __shared__ TileWalk s_walk;
    __shared__ int s_ok, s_chunk;
    const GemmLaunch &a = r.g;
    const int tiles_n = (a.N + T::BN - 1) / T::BN;
    const int rt_per_chunk = (a.rows_per_block + T::BM - 1) / T::BM;
    const int row_tiles = r.n_chunks * rt_per_chunk;
    const ListGrid lists(row_tiles, tiles_n, r.col_lists, r.group);
    auto total_of = [&](int x) { return lists.total(x); };

    if (threadIdx.x == 0) s_walk = TileWalk{0, 0, 0, 0, -1, 0, 0, 0};
    // Output streaming: a copy engine reads a piece of C while the kernel runs on, so
    // the tiles are written through the caches, and a tile is counted for its piece once every thread's
    // stores have been performed; whoever completes a piece lets its copy go. Ordering is by hand
    // (stores, their completion, barrier, counter, signal): a release fence would write back the whole
    // L2 once per tile. So that nobody waits for stores, a tile is counted under the next tile's
    // first k-step, or after the loop if it was the workgroup's last.
    int stored_chunk = -1;                 // thread 0: piece of the tile stored last and not yet counted
    auto count_stored = [&]() {
        if (STREAM_OUT && threadIdx.x == 0 && stored_chunk >= 0) {
            const uint32_t before = __hip_atomic_fetch_add(r.done_count + stored_chunk, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if ((before + 1u) % (uint32_t)r.tiles_per_chunk == 0u)
                __hip_atomic_store(reinterpret_cast<int64_t *>(r.done_sig[stored_chunk]), (int64_t)0, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_SYSTEM);
            stored_chunk = -1;
        }
    };
    for (;;) {
        if (threadIdx.x == 0) {
            TileWalk w = s_walk;
            tile_walk_next(w, r.ticket, r.ticket_base, r.grid, r.out, total_of);
            int ok = 1;
            if (w.x >= 0) {
                int R, tn;
                lists.position(w.x, w.t, R, tn);
                const int chunk = r.arrival[R / rt_per_chunk];
                if (chunk < r.local_chunk_begin || chunk >= r.local_chunk_end) ok = wait_ready(gate_argument(offsetof(ResidentLaunch, g.gate)), chunk, pace_of(r.grid, rt_per_chunk * tiles_n));
                s_chunk = chunk;           // the others take it from here instead of the table in memory
            }
            s_walk = w;
            s_ok = ok;
        }
        __syncthreads();                   // also orders the tile's loads after the flag read
        const int x = __builtin_amdgcn_readfirstlane(s_walk.x), t = __builtin_amdgcn_readfirstlane(s_walk.t);
        if (x < 0) break;
        if (s_ok) {
            int R, tn;
            lists.position(x, t, R, tn);
            const int rt = R % rt_per_chunk;
            const int chunk = __builtin_amdgcn_readfirstlane(s_chunk);
            const int64_t row0 = (int64_t)chunk * a.rows_per_block + (int64_t)rt * T::BM;
            const int rows_valid = min(T::BM, a.rows_per_block - rt * T::BM);
            const int col0 = tn * T::BN;
            const int cols_valid = min(T::BN, a.N - col0);
            TileAcc<T> ta;
            tile_zero(ta);
            if constexpr (STREAM_OUT)
                tile_accumulate<T>(ta, a.A + row0 * a.lda, rows_valid, a.Wt + (int64_t)col0 * a.K, cols_valid, a.lda, a.K, a.K, smem,
                                   count_stored);
            else
                tile_accumulate<T>(ta, a.A + row0 * a.lda, rows_valid, a.Wt + (int64_t)col0 * a.K, cols_valid, a.lda, a.K, a.K, smem);
            // the next ticket's round trip runs under the epilogue
            int have_drawn = 0;
            uint32_t drawn = 0;
            if (threadIdx.x == 0) have_drawn = tile_walk_predraw(s_walk, r.ticket, r.grid, r.out, total_of, drawn);
            if constexpr (STREAM_OUT) {
                tile_store<T, true>(ta, a.C + row0 * a.ldc + col0, rows_valid, cols_valid, a.ldc);
                stored_chunk = chunk;
            } else {
                tile_store<T>(ta, a.C + row0 * a.ldc + col0, rows_valid, cols_valid, a.ldc);
            }
            if (threadIdx.x == 0) { s_walk.have_drawn = have_drawn; s_walk.drawn = drawn; }
        }
        __syncthreads();                   // s_walk / s_ok / LDS stages are reused
    }
    wait_vmem<0>();                        // no load may arrive in LDS that is not this workgroup's any more; stores are done
    if constexpr (STREAM_OUT) {
        __syncthreads();
        count_stored();
    }
    leave_run(r.leave);
}

// Column-piece variant of the resident kernel (the 2D communication shape of Sec. V-A, chosen when
// M <= K): step s delivers K-slice s of every shard, and every tile of C can make progress at every
// step. The accumulation order over k is that of the monolithic kernel, so the bits are the same.
template <class T>
__global__ __launch_bounds__(T::THREADS) void gemm_resident2d_kernel(Resident2DLaunch r)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    __shared__ TileWalk s_walk;
    __shared__ int s_ok;
    const GemmLaunch &a = r.g;
    const int tiles_n = (a.N + T::BN - 1) / T::BN;
    const int row_tiles = (r.M + T::BM - 1) / T::BM;
    const ListGrid lists(row_tiles, tiles_n, r.col_lists, r.group);
    auto total_of = [&](int x) { return lists.total(x); };

    if (threadIdx.x == 0) s_walk = TileWalk{0, 0, 0, 0, -1, 0, 0, 0};
    for (;;) {
        if (threadIdx.x == 0) {
            TileWalk w = s_walk;
            tile_walk_next(w, r.ticket, r.ticket_base, r.grid, r.out, total_of);
            s_walk = w;
        }
        __syncthreads();
        const int x = __builtin_amdgcn_readfirstlane(s_walk.x), t = __builtin_amdgcn_readfirstlane(s_walk.t);
        if (x < 0) break;
        int tm, tn;
        lists.position(x, t, tm, tn);
        const int64_t row0 = (int64_t)tm * T::BM;
        const int rows_valid = min(T::BM, r.M - (int)row0);
        const int col0 = tn * T::BN;
        const int cols_valid = min(T::BN, a.N - col0);
        const int j0 = (int)(row0 / r.rows_per_shard), j1 = (int)((row0 + rows_valid - 1) / r.rows_per_shard);
        TileAcc<T> ta;
        tile_zero(ta);
        int ok = 1;
        // The k loop takes runs of slices: it waits for the next slice, then looks (without waiting) how many of
        // the following ones have landed as well, and multiplies the whole run as one k range, so that the load
        // pipeline is only drained where the kernel has to wait anyway. With operands resident the run is all of K.
        for (int sl = 0; sl < r.slices && ok;) {
            int run_end = r.slices;
            if (r.gated) {
                if (threadIdx.x < 64) {
                    const Gate gate = gate_argument(offsetof(Resident2DLaunch, g.gate));
                    const Pace pace = pace_of(r.grid, r.grid / r.shards);
                    const int o = wait_ready_all(gate, j1 - j0 + 1, pace, [&](int i) { return sl * r.shards + j0 + i; });
                    // one look at up to 64 following slices, a lane each
                    const int mine = sl + 1 + (int)threadIdx.x;
                    int landed = o && mine < r.slices;
                    for (int j = j0; j <= j1; ++j) landed = landed && peek_ready(gate, mine * r.shards + j, pace.every > 1, (poll_phase(blockIdx.x, pace.every) + sl) % pace.every == 0);
                    const uint64_t not_landed = ~__ballot(landed);
                    const int run = not_landed ? __builtin_ctzll(not_landed) : 64;
                    if (threadIdx.x == 0) s_ok = o ? sl + 1 + run : 0;      // 0: gave up; else the slice after the run
                }
                __syncthreads();           // also orders the run's loads after the flag reads
                run_end = s_ok;
                ok = run_end != 0;
                __syncthreads();
            }
            if (ok) {
                const int kb = r.k0[sl], ke = r.k0[run_end];              // the run's columns: [kb, ke)
                SlicedA<T> pa(a.A, r.k0, r.M, row0, sl, rows_valid, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), threadIdx.x & 63);
                tile_accumulate_from<T, NoHook, SlicedA<T>>(ta, pa, a.Wt + (int64_t)col0 * a.K + kb, cols_valid, a.K, ke - kb, smem);
                sl = run_end;
            }
        }
        int have_drawn = 0;
        uint32_t drawn = 0;
        if (threadIdx.x == 0) have_drawn = tile_walk_predraw(s_walk, r.ticket, r.grid, r.out, total_of, drawn);
        if (ok) tile_store<T>(ta, a.C + row0 * a.ldc + col0, rows_valid, cols_valid, a.ldc);
        if (threadIdx.x == 0) { s_walk.have_drawn = have_drawn; s_walk.drawn = drawn; }
        __syncthreads();                   // s_walk / s_ok / LDS stages are reused
    }
    wait_vmem<0>();                        // no load may arrive in LDS that is not this workgroup's any more
    leave_run(r.leave);
}

// Expert-parallel variant of the resident kernel (all-to-all token dispatch before the expert layers,
// Sec. II-A; unequal amounts per pair of GPUs, Sec. III-C): the rows of A are ragged segments, one per
// expert, each multiplied by that expert's weight. Row tiles never cross a segment; the host lists
// them in the order they become ready together with the pieces that cover them.
template <class T>
__global__ __launch_bounds__(T::THREADS) void gemm_grouped_kernel(GroupedLaunch r)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    __shared__ TileWalk s_walk;
    __shared__ int s_ok;
    const GemmLaunch &a = r.g;
    const int tiles_n = (a.N + T::BN - 1) / T::BN;
    const ListGrid lists(r.n_row_tiles, tiles_n, r.col_lists, r.group);
    auto total_of = [&](int x) { return lists.total(x); };

    if (threadIdx.x == 0) s_walk = TileWalk{0, 0, 0, 0, -1, 0, 0, 0};
    for (;;) {
        if (threadIdx.x < 64) {
            TileWalk w{};
            if (threadIdx.x == 0) {
                w = s_walk;
                tile_walk_next(w, r.ticket, r.ticket_base, r.grid, r.out, total_of);
                s_walk = w;
            }
            const int wx = __builtin_amdgcn_readfirstlane(w.x), wt = __builtin_amdgcn_readfirstlane(w.t);
            int ok = 1;
            if (wx >= 0 && r.gated) {
                int R, tn;
                lists.position(wx, wt, R, tn);
                const int32_t *rt = r.row_tiles + (size_t)R * kRowTileWords;
                const int first = rt[3];
                ok = wait_ready_all(gate_argument(offsetof(GroupedLaunch, g.gate)), rt[4] - first + 1, pace_of(r.grid, tiles_n), [&](int i) { return first + i; });
            }
            if (threadIdx.x == 0) s_ok = ok;
        }
        __syncthreads();                   // also orders the tile's loads after the flag reads
        const int x = __builtin_amdgcn_readfirstlane(s_walk.x), t = __builtin_amdgcn_readfirstlane(s_walk.t);
        if (x < 0) break;
        if (s_ok) {
            int R, tn;
            lists.position(x, t, R, tn);
            const int32_t *rt = r.row_tiles + (size_t)R * kRowTileWords;
            const int64_t row0 = rt[0];
            const int rows_valid = rt[1];
            const int64_t expert = rt[2];
            const int col0 = tn * T::BN;
            const int cols_valid = min(T::BN, a.N - col0);
            TileAcc<T> ta;
            tile_zero(ta);
            tile_accumulate<T>(ta, a.A + row0 * a.lda, rows_valid, a.Wt + (expert * a.N + col0) * (int64_t)a.K, cols_valid,
                               a.lda, a.K, a.K, smem);
            int have_drawn = 0;
            uint32_t drawn = 0;
            if (threadIdx.x == 0) have_drawn = tile_walk_predraw(s_walk, r.ticket, r.grid, r.out, total_of, drawn);
            tile_store<T>(ta, a.C + row0 * a.ldc + col0, rows_valid, cols_valid, a.ldc);
            if (threadIdx.x == 0) { s_walk.have_drawn = have_drawn; s_walk.drawn = drawn; }
        }
        __syncthreads();                   // s_walk / s_ok / LDS stages are reused
    }
    wait_vmem<0>();                        // no load may arrive in LDS that is not this workgroup's any more
}

__global__ __launch_bounds__(64) void wait_ready_kernel(Gate gate, const int32_t *chunks, int n)
{
    (void)wait_ready_all(gate, n, Pace{1, 1}, [&](int i) { return chunks[i]; });
}

// Nothing is published through the signal: what it orders is that the kernels before this one on the
// stream have finished reading A, which stream order has settled when this kernel starts. A relaxed store
// therefore does, and spares the cache write-back a release at system scope would add.
__global__ __launch_bounds__(64) void release_signal_kernel(int64_t *value)
{
    if (threadIdx.x == 0) __hip_atomic_store(value, (int64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// W[K,N] -> Wt[N,K], one wavefront per 64x64 tile, for a 16-byte aligned W, K % 64 == 0 and N % 8 == 0. A lane turns an
// 8x8 block in its registers (eight 16-byte loads, 32 byte permutes, eight 16-byte stores); lane l has k group l % 8 and
// column group l / 8, so that a load instruction reads, and a store instruction writes, whole 128-byte lines.
// Streaming work, bound by memory. The first workgroup also clears `clear_words` words at `clear` for the caller.
__global__ __launch_bounds__(256) void pack_weight_kernel(const uint16_t *__restrict__ W, uint16_t *__restrict__ Wt,
                                                          int64_t K, int64_t N, uint32_t *clear, int clear_words)
{
    if (blockIdx.x == 0 && blockIdx.y == 0 && (int)threadIdx.x < clear_words) clear[threadIdx.x] = 0u;
    const int lane = threadIdx.x & 63;
    const int64_t k0 = ((int64_t)blockIdx.y * 4 + (threadIdx.x >> 6)) * 64 + (lane & 7) * 8, n0 = (int64_t)blockIdx.x * 64 + (lane >> 3) * 8;
    if (k0 >= K || n0 >= N) return;
    u32x4_t r[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] = *reinterpret_cast<const u32x4_t *>(W + (k0 + i) * N + n0);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        u32x4_t even, odd;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            even[i] = __builtin_amdgcn_perm(r[2 * i + 1][c], r[2 * i][c], 0x05040100u);
            odd[i] = __builtin_amdgcn_perm(r[2 * i + 1][c], r[2 * i][c], 0x07060302u);
        }
        *reinterpret_cast<u32x4_t *>(Wt + (n0 + 2 * c) * K + k0) = even;
        *reinterpret_cast<u32x4_t *>(Wt + (n0 + 2 * c + 1) * K + k0) = odd;
    }
}

// The same for any W, 2 bytes at a time through a 64x64 LDS tile (padded), 256 threads.
__global__ __launch_bounds__(256) void pack_weight_unaligned_kernel(const uint16_t *__restrict__ W, uint16_t *__restrict__ Wt,
                                                                    int64_t K, int64_t N, uint32_t *clear, int clear_words)
{
    if (blockIdx.x == 0 && blockIdx.y == 0 && (int)threadIdx.x < clear_words) clear[threadIdx.x] = 0u;
    __shared__ uint16_t t[64][66];
    const int64_t k0 = (int64_t)blockIdx.y * 64, n0 = (int64_t)blockIdx.x * 64;
    for (int e = threadIdx.x; e < 64 * 64; e += 256) {
        int kk = e >> 6, nn = e & 63;
        if (k0 + kk < K && n0 + nn < N) t[kk][nn] = W[(k0 + kk) * N + n0 + nn];
    }
    __syncthreads();
    for (int e = threadIdx.x; e < 64 * 64; e += 256) {
        int nn = e >> 6, kk = e & 63;
        if (k0 + kk < K && n0 + nn < N) Wt[(n0 + nn) * K + k0 + kk] = t[kk][nn];
    }
}

// Sender-side re-layout of column pieces out of a row-major matrix (see SliceLaunch). 16-byte vectors, a row
// of a piece is width/8 of them; the workgroup's threads stride over (row, vector) pairs of its block.
__global__ __launch_bounds__(256) void slice_source_kernel(SliceLaunch a)
{
    // blocks in arrival order, a bounded number of workgroups striding over them: the pieces of the first step
    // are finished - and their transfers released - first instead of every piece at the end
    const int total_blocks = a.n_pieces * a.blocks_per_piece;
    for (int blk = blockIdx.x; blk < total_blocks; blk += gridDim.x) {
        const int q = blk / a.blocks_per_piece, b = blk % a.blocks_per_piece;
        const int piece = a.arrival[q];
        const int sl = piece / a.shards, j = piece % a.shards;
        const int kb = a.k0[sl], kw = a.k0[sl + 1] - kb;
        const int r0 = b * a.rows_per_block, r1 = min(a.rows_per_shard, r0 + a.rows_per_block);
        const int vecs = kw / 8;
        const u32x4_t *src = reinterpret_cast<const u32x4_t *>(a.src + ((int64_t)j * a.rows_per_shard + r0) * a.K + kb);
        u32x4_t *dst = reinterpret_cast<u32x4_t *>(a.dst + a.M * kb + ((int64_t)j * a.rows_per_shard + r0) * kw);
        const int64_t src_pitch = a.K / 8;
        const int total = (r1 - r0) * vecs;
        for (int e = threadIdx.x; e < total; e += 4 * 256) {
            u32x4_t v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int ee = e + u * 256;
                if (ee < total) v[u] = __builtin_nontemporal_load(src + (int64_t)(ee / vecs) * src_pitch + ee % vecs);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int ee = e + u * 256;
                // written through the caches: the reader is a copy engine
                if (ee < total) store_through_16(dst + ee, v[u]);
            }
        }
        // every store of the block has been performed (not just issued) before the block is counted
        wait_vmem<0>();
        __syncthreads();
        if (threadIdx.x == 0) {
            const uint32_t before = __hip_atomic_fetch_add(a.done_count + piece, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if ((before + 1u) % (uint32_t)a.blocks_per_piece == 0u)
                __hip_atomic_store(reinterpret_cast<int64_t *>(a.done_sig[piece]), (int64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

hipError_t launch_slice_source(const SliceLaunch &a, hipStream_t s)
{
    if (a.n_pieces <= 0 || a.blocks_per_piece <= 0 || a.rows_per_block <= 0) return hipErrorInvalidValue;
    const int64_t total = (int64_t)a.n_pieces * a.blocks_per_piece;
    if (total > 0x7FFFFFFF) return hipErrorInvalidValue;
    hipLaunchKernelGGL(slice_source_kernel, dim3((unsigned)std::min<int64_t>(total, 1024)), dim3(256), 0, s, a);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------ host
typedef TileCfg<256, 256, 2, 2, 2> T256x256;
typedef TileCfg<128, 128, 2, 2, 2> T128x128;       // two workgroups per CU: for launches that fill the machine
typedef TileCfg<128, 128, 2, 2, 4> T128x128D;      // deep ring, one workgroup per CU: for launches that do not
typedef TileCfg<256, 128, 2, 2, 3> T256x128;
typedef TileCfg<128, 256, 2, 2, 3> T128x256;
typedef TileCfg<64, 256, 1, 4, 3> T64x256;
typedef TileCfg<32, 256, 1, 4, 4> T32x256;
typedef TileCfg<128, 192, 2, 2, 3> T128x192;       // column counts that are multiples of 192 but not of 256
typedef TileCfg<256, 192, 2, 2, 2> T256x192;
// For launches that leave CUs idle with every larger tile. A CU draws 45-52 bytes a cycle from beyond its L2, about 32 when
// all of them do, whatever the tile, so a k-tile's time is its bytes: 24 KiB in 0.24-0.27 us here, 32 KiB in 0.31-0.40 with
// 128x128, and a short launch gains by spreading over more CUs. Six stages keep 120 KiB of loads in flight. M 1024, K 4096,
// N 768 30.6 -> 24.6 us.
typedef TileCfg<64, 128, 2, 2, 6> T64x128;
typedef TileCfg<64, 64, 2, 2, 8> T64x64;           // parts (is_part), rings of four and six pairs of stages
typedef TileCfg<32, 64, 2, 2, 12> T32x64;

// every tile shape, for the dispatch switches below
#define FICCO_FOR_EACH_TILE(X) \
    X(TILE_256x256, T256x256) X(TILE_128x128, T128x128) X(TILE_256x128, T256x128) X(TILE_128x256, T128x256) \
    X(TILE_64x256, T64x256) X(TILE_32x256, T32x256) X(TILE_128x128D, T128x128D) X(TILE_128x192, T128x192) \
    X(TILE_256x192, T256x192) X(TILE_64x128, T64x128) \
    X(TILE_64x64, T64x64) X(TILE_32x64, T32x64)

TileShape tile_shape(int tile)
{
    switch (tile) {
#define X(id, T) case id: return {T::BM, T::BN, T::LDS_BYTES, T::THREADS};
    FICCO_FOR_EACH_TILE(X)
#undef X
    default: return {0, 0, 0, 0};
    }
}

template <class T>
static hipError_t set_lds_limit(const void *fn)
{
    return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS_BYTES);
}

template <class T>
static hipError_t launch_gemm_t(const GemmLaunch &a, hipStream_t s)
{
    static hipError_t once = set_lds_limit<T>(reinterpret_cast<const void *>(&gemm_blocks_kernel<T>));
    if (once != hipSuccess) return once;
    const int tiles_n = (a.N + T::BN - 1) / T::BN;
    const int rt = (a.rows_per_block + T::BM - 1) / T::BM;
    const int64_t total = (int64_t)a.n_blocks * rt * tiles_n;
    if (total <= 0 || total > 0x7FFFFFFF || a.lda > kMaxK || a.K > kMaxK) return hipErrorInvalidValue;
    // at most as many workgroups as run at once (a multiple of 8, one share per XCD); the rest of the tiles
    // are taken by the kernel's loop
    int64_t grid = total;
    {
        static int fit_of[64];                       // per device: 0 = not asked yet, -1 = could not be asked
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess) return hipGetLastError();
        int fit = dev < 64 ? fit_of[dev] : 0;
        if (fit == 0) {
            int per_cu = 0, cus = 0;
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, gemm_blocks_kernel<T>, T::THREADS, T::LDS_BYTES) == hipSuccess &&
                hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && per_cu * cus >= 8)
                fit = per_cu * cus / 8 * 8;
            else
                fit = -1;
            if (dev < 64) fit_of[dev] = fit;
        }
        if (fit > 0 && total > fit) grid = fit;
    }
    // group height of the tile order: matters when the launch runs for several rounds
    GemmLaunch b = a;
    if (b.group_m != 1 && b.group_m != 2 && b.group_m != 4 && b.group_m != 8) b.group_m = 0;
    if (!b.group_m) b.group_m = 8;
    if (!a.group_m && total > grid) {
        double best = -1;
        for (int g = 1; g <= 8; g *= 2) {
            const double c = tile_order_cost(T::BM, T::BN, tiles_n, (int64_t)a.n_blocks * rt, grid / 8, 1, g,
                                             (int64_t)a.n_blocks * a.rows_per_block * a.K * 2, (int64_t)a.N * a.K * 2);
            if (best < 0 || c < best) { best = c; b.group_m = g; }
        }
    }
    hipLaunchKernelGGL(gemm_blocks_kernel<T>, dim3((unsigned)grid), dim3(T::THREADS), T::LDS_BYTES, s, b);
    return hipGetLastError();
}

template <class T>
static hipError_t launch_resident_t(const ResidentLaunch &r, hipStream_t s)
{
    static hipError_t once = set_lds_limit<T>(reinterpret_cast<const void *>(&gemm_resident_kernel<T, false>));
    static hipError_t once_out = set_lds_limit<T>(reinterpret_cast<const void *>(&gemm_resident_kernel<T, true>));
    if (once != hipSuccess) return once;
    if (once_out != hipSuccess) return once_out;
    if (r.grid <= 0 || r.g.lda > kMaxK || r.g.K > kMaxK) return hipErrorInvalidValue;
    if (r.done_count)
        hipLaunchKernelGGL((gemm_resident_kernel<T, true>), dim3((unsigned)r.grid), dim3(T::THREADS), T::LDS_BYTES, s, r);
    else
        hipLaunchKernelGGL((gemm_resident_kernel<T, false>), dim3((unsigned)r.grid), dim3(T::THREADS), T::LDS_BYTES, s, r);
    return hipGetLastError();
}

template <class T>
static hipError_t launch_resident2d_t(const Resident2DLaunch &r, hipStream_t s)
{
    static hipError_t once = set_lds_limit<T>(reinterpret_cast<const void *>(&gemm_resident2d_kernel<T>));
    if (once != hipSuccess) return once;
    if (r.grid <= 0 || !r.k0 || r.g.K > kMaxK) return hipErrorInvalidValue;
    hipLaunchKernelGGL(gemm_resident2d_kernel<T>, dim3((unsigned)r.grid), dim3(T::THREADS), T::LDS_BYTES, s, r);
    return hipGetLastError();
}

template <class T>
static int resident2d_grid_t(int device)
{
    static hipError_t once = set_lds_limit<T>(reinterpret_cast<const void *>(&gemm_resident2d_kernel<T>));
    (void)once;
    int per_cu = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, gemm_resident2d_kernel<T>, T::THREADS, T::LDS_BYTES) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) return 0;
    return per_cu * cus;
}

template <class T>
static hipError_t launch_grouped_t(const GroupedLaunch &r, hipStream_t s)
{
    static hipError_t once = set_lds_limit<T>(reinterpret_cast<const void *>(&gemm_grouped_kernel<T>));
    if (once != hipSuccess) return once;
    if (r.grid <= 0 || r.n_row_tiles <= 0 || r.g.lda > kMaxK || r.g.K > kMaxK) return hipErrorInvalidValue;
    hipLaunchKernelGGL(gemm_grouped_kernel<T>, dim3((unsigned)r.grid), dim3(T::THREADS), T::LDS_BYTES, s, r);
    return hipGetLastError();
}

template <class T>
static int grouped_grid_t(int device)
{
    static hipError_t once = set_lds_limit<T>(reinterpret_cast<const void *>(&gemm_grouped_kernel<T>));
    (void)once;
    int per_cu = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, gemm_grouped_kernel<T>, T::THREADS, T::LDS_BYTES) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) return 0;
    return per_cu * cus;
}

template <class T>
static int resident_grid_t(int device)
{
    static hipError_t once = set_lds_limit<T>(reinterpret_cast<const void *>(&gemm_resident_kernel<T, false>));
    (void)once;
    int per_cu = 0, cus = 0;
    // (the output-streaming form may need more registers, but every tile shape is limited by LDS first)
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, gemm_resident_kernel<T, false>, T::THREADS, T::LDS_BYTES) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) return 0;
    return per_cu * cus;
}


hipError_t launch_gemm(int tile, const GemmLaunch &a, hipStream_t s)
{
    switch (tile) {
#define X(id, T) case id: return launch_gemm_t<T>(a, s);
    FICCO_FOR_EACH_TILE(X)
#undef X
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_resident(int tile, const ResidentLaunch &r, hipStream_t s)
{
    switch (tile) {
#define X(id, T) case id: return launch_resident_t<T>(r, s);
    FICCO_FOR_EACH_TILE(X)
#undef X
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_resident2d(int tile, const Resident2DLaunch &r, hipStream_t s)
{
    switch (tile) {
#define X(id, T) case id: return launch_resident2d_t<T>(r, s);
    FICCO_FOR_EACH_TILE(X)
#undef X
    default: return hipErrorInvalidValue;
    }
}

int resident2d_grid_size(int tile, int device)
{
    switch (tile) {
#define X(id, T) case id: return resident2d_grid_t<T>(device);
    FICCO_FOR_EACH_TILE(X)
#undef X
    default: return 0;
    }
}

int resident_grid_size(int tile, int device)
{
    switch (tile) {
#define X(id, T) case id: return resident_grid_t<T>(device);
    FICCO_FOR_EACH_TILE(X)
#undef X
    default: return 0;
    }
}

hipError_t launch_wait_ready(const Gate &gate, const int32_t *chunks, int n, hipStream_t s)
{
    hipLaunchKernelGGL(wait_ready_kernel, dim3(1), dim3(64), 0, s, gate, chunks, n);
    return hipGetLastError();
}

hipError_t launch_release_signal(uint64_t value_addr, hipStream_t s)
{
    if (!value_addr) return hipErrorInvalidValue;
    hipLaunchKernelGGL(release_signal_kernel, dim3(1), dim3(64), 0, s, reinterpret_cast<int64_t *>(value_addr));
    return hipGetLastError();
}

hipError_t launch_pack_weight(const uint16_t *W, uint16_t *Wt, int64_t K, int64_t N, hipStream_t s, uint32_t *clear, int clear_words)
{
    if (clear_words < 0 || clear_words > 256) return hipErrorInvalidValue;
    const unsigned tn = (unsigned)((N + 63) / 64);
    if ((uintptr_t)W % 16 == 0 && (uintptr_t)Wt % 16 == 0 && K % 64 == 0 && N % 8 == 0)
        hipLaunchKernelGGL(pack_weight_kernel, dim3(tn, (unsigned)((K + 255) / 256)), dim3(256), 0, s, W, Wt, K, N, clear, clear_words);
    else
        hipLaunchKernelGGL(pack_weight_unaligned_kernel, dim3(tn, (unsigned)((K + 63) / 64)), dim3(256), 0, s, W, Wt, K, N, clear, clear_words);
    return hipGetLastError();
}

hipError_t launch_grouped(int tile, const GroupedLaunch &r, hipStream_t s)
{
    switch (tile) {
#define X(id, T) case id: return launch_grouped_t<T>(r, s);
    FICCO_FOR_EACH_TILE(X)
#undef X
    default: return hipErrorInvalidValue;
    }
}

int grouped_grid_size(int tile, int device)
{
    switch (tile) {
#define X(id, T) case id: return grouped_grid_t<T>(device);
    FICCO_FOR_EACH_TILE(X)
#undef X
    default: return 0;
    }
}

}  // namespace ficco
