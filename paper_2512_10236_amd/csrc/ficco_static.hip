// ficco_gemm_static: the GEMM over operands that are already in place (small products straight from the row-major
// weight, others by the resident kernel), for callers that cannot allocate device memory (code under HIP graph capture, tight serving loops, harnesses that
// forbid hipMalloc). Everything the resident kernel needs beyond its inputs and outputs - the ticket
// counters of its tile lists, the status word of its bounded waits, the one-entry arrival table and
// the packed copy of the weight - lives in one file-scope device array instead of plan-owned
// allocations. See include/ficco.h for the contract.
#include "ficco_plan.h"

namespace ficco {
namespace {

constexpr size_t kHeadBytes = 4096;                                  // counters, status word, arrival table
constexpr size_t kStaticBytes = kHeadBytes + FICCO_STATIC_MAX_WEIGHT_BYTES;
// layout of the head, in 32-bit words: [0, 144) ticket counters (kTicketLists + 1 lines of 16 words),
// [160] status word, [176] arrival table (one entry)
constexpr int kStatusWord = 160, kArrivalWord = 176, kHeadWordsCleared = 192;

// Every GPU the library runs on holds its own copy of this array until the process ends. Host code
// never passes the array's name to a kernel or a copy: the name is a host-side stand-in, and the
// address of a device's copy comes from hipGetSymbolAddress (scratch_of below).
static __device__ __align__(256) unsigned char scratch[kStaticBytes];

unsigned char *g_scratch_of[64];                                      // per device, filled on first use

int scratch_of(int dev, unsigned char **out)
{
    if (dev < 0 || dev >= 64) return FICCO_ERR_ARG;
    if (!g_scratch_of[dev]) {
        void *ptr = nullptr;
        HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));       // the current device's copy
        if (!ptr) return FICCO_ERR_HIP;
        g_scratch_of[dev] = static_cast<unsigned char *>(ptr);
    }
    *out = g_scratch_of[dev];
    return FICCO_OK;
}

}  // namespace

// Which way a call goes: 0 = pack the weight, then the resident GEMM; else one launch of the direct kernel on tiles of
// 16 * row_blocks rows x 64 columns. The direct kernel needs no packed weight but fetches every operand row once per
// narrow tile, so it wins where a launch is a round or two of its tiles and loses where the resident kernel's big tiles
// fill the chip. Estimates in us, from timings over M 1-8192, K 64-8192, N 8-4096: a stage of 128 k values takes 0.25 /
// 0.31 / 0.46 us with 1 / 2 / 4 row blocks, a round starts in 2 us; the packed way takes the tile rule's estimate and 6 us
// for the packing launch (3.9) and the gap behind it. Over 600 random products (M 1-8192, K 512-8192, N 64-4096) the way
// taken is 0.1 % slower than the fastest (0.4 with 0.55, 1.5 and 4 in the place of 0.46, 2 and 6; calls under 4.6 us, which
// the host takes, count as that). Measured, direct against packed: M 576, K 4224, N 992 16.3 : 22.7, M 1225, K 2496, N 904
// 22.0 : 20.9, M 1596, K 1600, N 1880 27.3 : 21.5, M 2594, K 4096, N 680 39.6 : 27.4.
int direct_row_blocks(int64_t M, int64_t K, int64_t N, int cus, double packed_us)
{
    static const struct { int row_blocks; double stage; } cand[] = {{1, 0.25}, {2, 0.31}, {4, 0.46}};
    double best = packed_us + 6.0;
    int best_id = 0;
    for (auto &cd : cand) {
        const int64_t tiles = ((M + 16 * cd.row_blocks - 1) / (16 * cd.row_blocks)) * ((N + 63) / 64);
        const double t = (double)((tiles + cus - 1) / cus) * (2.0 + cd.stage * (double)((K + 127) / 128)) + 2.0;
        if (t < best) { best = t; best_id = cd.row_blocks; }
    }
    return best_id;
}

}  // namespace ficco

using namespace ficco;

extern "C" int ficco_gemm_static(int64_t M, int64_t K, int64_t N, const void *A_dev, const void *W_dev, void *C_dev, void *stream)
{
    if (!A_dev || !W_dev || !C_dev) return FICCO_ERR_ARG;
    if (M < 1 || K < 1 || N < 1 || K % 64 || N % 8 || M > 0x7FFFFFFF || N > 0x7FFFFFFF || K > kMaxK) return FICCO_ERR_SHAPE;
    if ((uint64_t)K * (uint64_t)N * 2u > (uint64_t)FICCO_STATIC_MAX_WEIGHT_BYTES) return FICCO_ERR_SHAPE;
    bool dev_ptr = false;
    for (const void *ptr : {A_dev, W_dev, (const void *)C_dev}) {
        int rc = is_device_ptr(ptr, &dev_ptr);
        if (rc || !dev_ptr) return FICCO_ERR_ARG;
    }
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    unsigned char *base = nullptr;
    int rc = scratch_of(dev, &base);
    if (rc) return rc;
    uint32_t *head = reinterpret_cast<uint32_t *>(base);
    uint16_t *wt = reinterpret_cast<uint16_t *>(base + kHeadBytes);
    hipStream_t s = (hipStream_t)stream;
    // the shape as a one-piece resident plan (host-side bookkeeping only): same tile choice and tile order
    // as ficco_run gives such a plan, hence the same kernel
    ficco_plan_t shape;
    shape.M = M; shape.K = K; shape.N = N; shape.G = 1; shape.c = 1;
    shape.schedule = FICCO_FINE_PERSISTENT;
    shape.order = FICCO_ORDER_STEP_MAJOR;
    shape.mode = FICCO_MODE_GEMM_ONLY;
    if ((rc = build_lists(&shape))) return rc;
    int cus = 0;
    HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    double packed_us = 0;
    // A weight that is not 16-byte aligned, or that the result overwrites, is packed first. A result over the activation
    // needs it too: the direct kernel's tiles are narrower than most outputs, and while one stores, another still reads
    // the same rows of A. The packed way then takes a tile as wide as the output.
    const bool over_a = overlap(C_dev, 2 * M * N, A_dev, 2 * M * K);
    shape.tile = choose_tile(&shape, cus, over_a, &packed_us);
    const bool packed_only = over_a || (uintptr_t)W_dev % 16 || overlap(C_dev, 2 * M * N, W_dev, 2 * K * N);
    const int row_blocks = packed_only ? 0 : direct_row_blocks(M, K, N, cus, packed_us);
    if (row_blocks) {
        DirectLaunch d{};
        d.A = (const uint16_t *)A_dev;
        d.W = (const uint16_t *)W_dev;
        d.C = (uint16_t *)C_dev;
        d.M = (int32_t)M; d.N = (int32_t)N; d.K = (int32_t)K;
        HIP_TRY(launch_direct(row_blocks, d, s));
        return FICCO_OK;
    }
    const TileShape ts = tile_shape(shape.tile);
    if (ts.bm == 0) return FICCO_ERR_ARG;
    const int64_t row_tiles = (M + ts.bm - 1) / ts.bm, tn = (N + ts.bn - 1) / ts.bn;
    int grid = resident_grid_size(shape.tile, dev);
    if (grid <= 0) return FICCO_ERR_HIP;
    if (row_tiles * tn < grid) grid = (int)(row_tiles * tn);
    shape.resident_grid = grid;
    const ListGeometry lg = resident_lists(&shape);
    if (!lg.col_lists) return FICCO_ERR_ARG;
    int khz = 100000;
    (void)hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev);

    // The array keeps the last call's contents: counters, status and the arrival entry start every call from zero, which
    // the packing kernel sees to (no memset, so that a caller may capture the call into a graph).
    HIP_TRY(launch_pack_weight((const uint16_t *)W_dev, wt, K, N, s, head, kHeadWordsCleared));

    ResidentLaunch r{};
    r.g.A = (const uint16_t *)A_dev;
    r.g.Wt = wt;
    r.g.C = (uint16_t *)C_dev;
    r.g.lda = K;
    r.g.ldc = N;
    r.g.N = (int32_t)N;
    r.g.K = (int32_t)K;
    r.g.n_blocks = 1;
    r.g.rows_per_block = (int32_t)M;
    r.g.group_m = 0;
    // nothing is waited for (the one piece is resident); the gate only has to point at valid words
    r.g.gate = Gate{head + kStatusWord + 4, nullptr, 1u, head + kStatusWord, head + kStatusWord, (uint64_t)khz * 2000u};
    r.arrival = reinterpret_cast<const int32_t *>(head + kArrivalWord);
    r.n_chunks = 1;
    r.ticket = head;
    for (int x = 0; x < kTicketLists; ++x) r.ticket_base[x] = 0;      // the counters were just cleared
    r.grid = grid;
    r.group = lg.group;
    r.col_lists = lg.col_lists;
    r.out = hand_out(row_tiles, tn, lg.col_lists, grid, false);
    r.local_chunk_begin = 0;
    r.local_chunk_end = 1;
    HIP_TRY(launch_resident(shape.tile, r, s));
    return FICCO_OK;
}
