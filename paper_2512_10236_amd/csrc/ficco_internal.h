// Internal declarations shared by the kernel file and the C-ABI file of libficco. Not installed.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stddef.h>
#include <stdint.h>

namespace ficco {

// Workgroup tile shapes. The k order (ascending, 32 at a time inside one 16x16x32 MFMA) is the
// same in all of them, so the output bits do not depend on the choice.
enum TileId : int { TILE_256x256 = 1, TILE_128x128 = 2, TILE_256x128 = 3, TILE_128x256 = 4,
                    TILE_64x256 = 5, TILE_32x256 = 6, TILE_128x128D = 7, TILE_128x192 = 8, TILE_256x192 = 9,
                    TILE_64x128 = 10, TILE_64x64 = 11, TILE_32x64 = 12, TILE_COUNT = 13 };

// The last two are parts that a launch's tiles are cut into, a workgroup each, where that is faster than whole ones (few
// tiles, CUs idle).
inline bool is_part(int tile) { return tile == TILE_64x64 || tile == TILE_32x64; }

struct TileShape { int bm, bn, lds_bytes, threads; };
TileShape tile_shape(int tile);

constexpr int kFlagStrideWords = 16;      // one ready flag per 64-byte line
constexpr int kBK = 64;                   // k extent of one LDS stage
// Largest K (row stride of A and of the packed weight, in elements): the loaders address a tile's rows with 32-bit
// byte offsets from a 64-bit base, and 256 rows of 2^22 elements of 2 bytes span 2 GiB.
constexpr int64_t kMaxK = (int64_t)1 << 22;
constexpr int kTicketLists = 8;           // one tile list per XCD (each XCD has its own L2)

// Tiles of the resident kernels that list x (of kTicketLists) holds. The lists form a grid of
// kTicketLists / col_lists row classes by col_lists column blocks: list x takes the row tiles
// rc, rc + classes, rc + 2 classes, ... (rc = x % classes) of the arrival-ordered sequence of row
// tiles, times the column tiles of block x / classes (the column tiles cut into col_lists nearly
// equal runs). col_lists = 1: every list spans all column tiles.
__host__ __device__ inline int64_t resident_list_tiles(int64_t row_tiles, int64_t tiles_n, int x, int col_lists = 1)
{
    const int classes = kTicketLists / col_lists, rc = x % classes, cb = x / classes;
    const int64_t rows = row_tiles > rc ? (row_tiles - rc + classes - 1) / classes : 0;
    return rows * ((cb + 1) * tiles_n / col_lists - cb * tiles_n / col_lists);
}

// Relative cost of a tile order for one XCD, whose L2 is filled with what its workgroups have in
// flight: `slots` tiles taken from groups of g row tiles x `width` column tiles (width = the tn column
// tiles cut into col_lists blocks), i.e. part of one group or several whole groups. Counted in operand
// rows per k-step - rows of A plus rows of the packed weight - each weighted by where the fill comes
// from: the memory-side cache costs 1, HBM costs kHbmFillCost, and the kernels, whose rings hold two or
// three k-steps, feel that latency. A line is fetched from HBM by the first XCD that wants it; the
// XCDs that walk the same rows (the col_lists lists of a row class) or the same columns (the
// kTicketLists / col_lists lists of a column block) at the same time find it in the cache, and so do
// later passes over a group's rows and later groups' passes over the columns if the operand stays
// there (operands up to kCacheStayBytes do; a group's rows also do between its own rounds when the
// rows all row classes hold at that time fit). Among equal footprints groups of about three rounds of
// tiles were fastest. Fitted to sweeps of all 16 (col_lists, g) pairs on five shape/tile combinations
// (14 to 112 column tiles, 16 to 128 row tiles, 128x128 and 256x256 tiles) and checked against such
// sweeps on 8 shapes x 3 launch kinds: the pick is within 2 % of the best order in 23 of 24 cases.
// Known miss: with 128-row pieces of a short, very wide product (M = 4096, N = 14336) and the
// 128x128 tile (no longer chosen for it) the orders a step-bound group allows are all 6-16 % slower
// than the best free order, and the model picks the slowest of them.
constexpr double kHbmFillCost = 3.0;
constexpr int64_t kCacheStayBytes = 128ll << 20;       // of the 256 MB memory-side cache
__host__ inline double tile_order_cost(int bm, int bn, int64_t tn, int64_t row_tiles, int64_t slots, int col_lists, int g,
                                       int64_t a_bytes, int64_t w_bytes)
{
    const int classes = kTicketLists / col_lists;
    const int64_t rows_list = row_tiles / classes > 1 ? (row_tiles + classes - 1) / classes : 1;
    if (g > rows_list) g = (int)rows_list;
    const int64_t width = (tn + col_lists - 1) / col_lists;
    const int64_t per_group = (int64_t)g * width;
    const double rows_active = per_group >= slots ? (double)g : (double)g * (double)slots / (double)per_group;
    double cols_active = (double)slots / g > 1.0 ? (double)slots / g : 1.0;
    if (cols_active > (double)width) cols_active = (double)width;
    const double passes = per_group > slots ? (double)per_group / (double)slots : 1.0;       // rounds a group's rows stay in use
    const double groups = rows_list > g ? (double)rows_list / g : 1.0;                       // passes over a list's columns
    // a group's rows are needed for `passes` rounds in a row: the later ones find them cached if the rows that
    // all row classes hold at that time fit, even when the whole of A does not
    const int64_t group_rows_bytes = row_tiles > 0 ? a_bytes / row_tiles * g * classes : a_bytes;
    const double a_from_hbm = (a_bytes <= kCacheStayBytes || group_rows_bytes <= kCacheStayBytes) ? 1.0 / (col_lists * passes) : 1.0 / col_lists;
    const double w_from_hbm = w_bytes <= kCacheStayBytes ? 1.0 / (classes * groups) : 1.0 / classes;
    const double fill = rows_active * bm * (1.0 + (kHbmFillCost - 1.0) * a_from_hbm) +
                        cols_active * bn * (1.0 + (kHbmFillCost - 1.0) * w_from_hbm);
    const double off = log2((double)per_group / (3.0 * (double)slots));
    return fill * (1.0 + 0.02 * (off < 0 ? -off : off));
}

// Workgroups of a resident launch whose first list is x (workgroup b starts on list b % kTicketLists).
__host__ __device__ inline int resident_list_homes(int grid, int x) { return grid > x ? (grid - x + kTicketLists - 1) / kTicketLists : 0; }

// How a resident launch hands out its tiles. A draw from a list's counter is a round trip of 3-4 us to memory that all
// XCDs share, and at the end of a launch every workgroup makes one on every list that has counters in use. So:
//   short launches (by_rank) use no counters. A workgroup has `rounds` places on its home list, rank, rank + homes, rank +
//     2 homes, ... Where the list is shorter than its places, the spare ones, counted over all lists, take the tiles that the
//     longer lists have too many, counted the same way (tile_by_rank). There are always enough: rounds * grid >= all tiles.
//   longer ones let workgroups drift apart: the first three quarters of a workgroup's share of its home list go by rank,
//     or one tile where the lists are uneven, and the rest is drawn (tile_walk_next).
// By rank instead of by draws, even lists: M 2048, K 1024, N 4096 45.7 -> 34.6 us, M 9600, K 512, N 256 17.0 -> 13.7; uneven
// ones: M 2654, K 640, N 3008 40.4 -> 18.0, M 7397, K 320, N 3088 58.0 -> 28.6. The line between the two, launches of 9 to 16
// tiles a workgroup by rank against by draws: M 19089, K 128, N 4144 54.9 : 94.5, M 16384, K 1024, N 10240 333 : 346, M 20480,
// K 2048, N 9216 643 : 633, M 12288, K 4096, N 16384 and M 16384, K 8192, N 9728 the same.
// Where tiles wait for pieces (waits), a workgroup that is held up by a late piece must not hold a second tile that another
// one could take: uneven lists go by rank only where every workgroup has one place (pairs and experts of two to five rounds
// by rank against by draws: M 7936, K 14080, N 6216 2264 : 2134, experts 5922x6400x2816 547 : 515, 22858x4928x1744 1080 : 1038),
// even ones up to 8.
constexpr int kStaticRounds = 16, kStaticRoundsWaiting = 8;
struct HandOut { int rounds, by_rank; };
__host__ inline HandOut hand_out(int64_t row_tiles, int64_t tiles_n, int col_lists, int grid, bool waits)
{
    int64_t most = 1, total = 0;
    bool all_started = true;
    for (int x = 0; x < kTicketLists; ++x) {
        const int64_t t = resident_list_tiles(row_tiles, tiles_n, x, col_lists), h = resident_list_homes(grid, x);
        total += t;
        if (t > 0 && h == 0) all_started = false;           // a list nobody starts on
        if (h > 0 && (t + h - 1) / h > most) most = (t + h - 1) / h;
    }
    const int64_t even = (total + grid - 1) / grid;
    const bool evenly = all_started && most <= even;
    if (even <= (!waits ? kStaticRounds : evenly ? kStaticRoundsWaiting : 1)) return {(int)even, 1};
    return {(int)(evenly ? even * 3 / 4 : 1), 0};
}

// by_rank: the tile of place `taken` of the workgroup of this rank on list `home`; false: none, nor any further on.
template <class TotalFn>
__host__ __device__ inline bool tile_by_rank(int home, int rank, int taken, int grid, int rounds, TotalFn total_of, int &x, int &t)
{
    const int place = rank + taken * resident_list_homes(grid, home), total = total_of(home);
    if (place < total) { x = home; t = place; return true; }
    int spare = place - total;
#pragma unroll 1
    for (int k = 0; k < home; ++k) {
        const int left = rounds * resident_list_homes(grid, k) - total_of(k);
        if (left > 0) spare += left;
    }
#pragma unroll 1
    for (int k = 0; k < kTicketLists; ++k) {
        const int places = rounds * resident_list_homes(grid, k), over = total_of(k) - places;
        if (over <= 0) continue;
        if (spare < over) { x = k; t = places + spare; return true; }
        spare -= over;
    }
    return false;
}

// Atomic draws one resident launch makes on list x's counter: none by rank, nor if the ranks of its own workgroups cover
// the list; otherwise every later tile is drawn and every workgroup draws exactly one ticket past the end of the list. The
// host advances its copy of each counter by this much per launch, so counters are never reset.
__host__ __device__ inline uint32_t resident_list_draws(int64_t list_tiles, int grid, int x, HandOut h)
{
    const int64_t taken = (int64_t)h.rounds * resident_list_homes(grid, x);
    return !h.by_rank && list_tiles > taken ? (uint32_t)(list_tiles - taken + grid) : 0u;
}

// How a kernel learns that piece `chunk` has landed:
//   flags     - flags[chunk*kFlagStrideWords] == epoch (a 4-byte copy or stream write queued behind the transfer)
//   sig_value - the 64-bit word at sig_value[chunk] has dropped to 0: the value field of the transfer's
//               own completion signal, decremented by the copy engine itself
// Both are read at system scope; the wait is bounded (status[0] = 1 when it expires).
// The signals' words lie in host memory, and what reads them shares the host link with the engines' own writes to them. So
// where many workgroups wait, each looks there on some of its polls only (pace_of), passes on what it sees landed - the
// run's epoch, into the piece's flag in device memory, which no transfer writes then - and watches that flag on all others.
constexpr uint32_t kRunTag = 0x80000000u;
struct Gate {
    uint32_t *flags;              // one for each signal of the table
    const uint64_t *sig_value;    // device table of addresses, or nullptr to use flags
    uint32_t epoch;               // of the run; with signals kRunTag | its number, which no flag copy and no earlier run writes
    uint32_t *status;             // device word every waiting workgroup watches
    uint32_t *status_host;        // pinned host word set together with it, so that the host needs no copy to see it
    uint64_t spin_limit_ticks;    // in wall_clock64() ticks
};
// How a workgroup waits, of `workgroups` that wait and `same` of them for the same piece. It looks at the signals on one of
// `every` polls: about four of those that wait for a piece look at a time, and about 32 of all (1: on every poll, and nothing
// is passed on). With all of them looking all the time each costs a launch about 0.1 us; four a piece see it land as soon as
// all would (us a pass, all / 8 / 4 / 2 of those at a time: M 4096, K 2048, N 256 over eight shards, 256 workgroups of 64x64
// tiles, 32 a piece 76.0 / - / 73.2 / 75.7; M 512, K 1024, N 1024 over four shards, 256 workgroups of 32x64, 64 a piece 41.2 /
// 37.5 / 35.3 / -; one launch per step, M 4096, K 8192, N 3584, 224 workgroups, all / 28 of them at eight signals 355.8 / 330.7).
// A flag that hundreds of workgroups read as fast as they can holds up what else goes to that place in memory: from about
// a hundred on a piece, polls are `naps` times as far apart (the same launches per step at 1 / 4 / 12 naps 315 / 308 / 303, M
// 4096, K 2048, N 2048 122 / 116 / 108; with 64 a piece they only see it later, 44.5 / 47.2 / 47.1 at M 512).
struct Pace { uint32_t every, naps; };
__device__ inline Pace pace_of(uint32_t workgroups, uint32_t same)
{
    if (same > workgroups) same = workgroups;
    const uint32_t n = same / 4 > workgroups / 32 ? same / 4 : workgroups / 32;
    return {n < 1 ? 1 : n > 16 ? 16 : n, same < 96 ? 1 : same / 24};
}
// Where a workgroup's looks at the signals lie among its polls. Those that wait for the same piece are of one list of tiles
// (workgroup b is at home in list b % kTicketLists) or of all of them: the rank in the list tells them apart, and the lists
// start an eighth of the interval one behind the other, so that few ranks are spread over it too. (All behind eight shards,
// M 2048, K 192, N 2048: 43.7 us a pass with the number itself, which has those of one XCD look together, 40.4 this way.)
__host__ __device__ inline uint32_t poll_phase(uint32_t workgroup, uint32_t every)
{
    return workgroup / kTicketLists + workgroup % kTicketLists * every / kTicketLists;
}
// What a wavefront that waits for several pieces looks at on each of its polls: on one of `every` at the signal of the last
// one that is missing (pieces are listed in the order in which they leave), on all others at its flag alone. When it has
// landed the poll behind it is at all flags, and the next look at the signals is a wide one, at those of the kLookWide last missing
// pieces (of all, where few workgroups wait and `every` is 1); so is every kLookEvery-th, and each where no more than kLookFew
// pieces are missing. Before it gives up it looks at everything. Pieces that have landed before a wait thus cost it one interval for each kLookWide of them and one more, also where
// nobody else passes them on.
// Wide looks are dear where hundreds of workgroups have them at the same time (us a pass; on the first poll of every wait / on
// the poll behind a landing / this way: launches per step, M 8192, K 1024, N 1024 over eight shards of four pieces 222 / 124 /
// 116; all of M 2048, K 192, N 2048 behind eight shards 69 / 42 / 41), and so are wider ones (at all missing pieces: eight
// experts, four steps, 32 pieces a tile, M 1675, K 3264, N 7496 514 against 508).
constexpr uint32_t kLookEvery = 8, kLookFew = 2, kLookWide = 8;
struct PollPlan {
    uint32_t every, polls, looks, wide;
    uint32_t signals;              // this poll: at the signals of that many of the missing pieces, from the last one down ...
    int flags = 1;                 // ... and at the flags of all of them, or of the last one
    int again = 0;                 // the next look is a wide one
    __host__ __device__ PollPlan(uint32_t every_, uint32_t phase)
        : every(every_), polls(phase), looks(0), wide(every_ == 1 ? 64 : kLookWide), signals(phase % every_ == 0 ? wide : 0) {}
    // last_landed: the last one that was missing has; late: the limit is over; missing: pieces
    __host__ __device__ void next(int last_landed, int late, uint32_t missing)
    {
        const int turn = ++polls % every == 0, few = missing <= kLookFew;
        looks += (uint32_t)turn;
        again |= last_landed;
        signals = late ? 64 : !turn ? 0 : few || again || looks % kLookEvery == 0 ? wide : 1;
        if (turn) again = 0;
        flags = last_landed || late || few || signals > 1;
    }
};

// One GEMM launch over a list of equal-height row blocks of A/C (one block for a monolithic or
// per-piece launch, G blocks for a fused step).
struct GemmLaunch {
    const uint16_t *A;        // [*, K] bf16, leading dimension lda
    const uint16_t *Wt;       // packed weight [N, K] bf16
    uint16_t *C;              // [*, N] bf16, leading dimension ldc
    int64_t lda, ldc;
    int32_t N, K;
    const int32_t *block_row0;   // device table of n_blocks first rows, or nullptr
    int32_t row0;                // first row when block_row0 == nullptr (n_blocks == 1)
    int32_t n_blocks;
    int32_t rows_per_block;
    int32_t group_m;             // row tiles per group of the tile order: 1, 2, 4, 8, or 0 = the launcher chooses
    // Optional gate (copy-engine transfers): every workgroup waits until all of the pieces
    // wait_chunks[0..n_wait) are ready.
    Gate gate;
    const int32_t *wait_chunks;
    int32_t n_wait;
};

// What a resident kernel does on its way out when other plans' transfers wait for the end of this run
// (chained plans): every workgroup counts itself out, and the one that brings the counter (device,
// never reset) to `target` stores 0 into the value word of the signal those transfers depend on.
// release_value == nullptr: nothing to do.
struct RunExit {
    uint32_t *count;
    uint32_t target;
    int64_t *release_value;
};

// The resident kernel: tiles are taken from a ticket counter in arrival order; the tiles of the
// piece issued p-th wait until that piece is ready (g.gate).
struct ResidentLaunch {
    GemmLaunch g;                 // block_row0/row0/n_blocks/wait_chunks unused; rows_per_block = piece rows
    const int32_t *arrival;       // device, n_chunks chunk ids in arrival order
    int32_t n_chunks;
    uint32_t *ticket;             // device, kTicketLists counters kFlagStrideWords apart, monotonically increasing across runs
    uint32_t ticket_base[8];      // value of each counter when this run starts
    int32_t grid;                 // workgroups
    HandOut out;
    int32_t group;                // row tiles per group of a list's tile order (1..8)
    int32_t col_lists;            // column blocks the lists are split into (1, 2, 4 or 8; see resident_list_tiles)
    int32_t local_chunk_begin, local_chunk_end;   // chunk ids that need no flag (already resident), or empty
    // GEMM -> reduce-scatter: when the last tile of a piece has been stored, the kernel releases the copy
    // that waits for the piece by storing 0 into the value word of the copy's dependency signal.
    uint32_t *done_count;         // device, one counter per chunk id, never reset: a run adds tiles_per_chunk to each
    const uint64_t *done_sig;     // device table: address of the value word of each chunk's dependency signal
    int32_t tiles_per_chunk;      // row tiles per piece x column tiles
    RunExit leave;
};

// The resident kernel for column (K) pieces: A is kept in K-sliced layout, slice after slice, slice s
// being the [M][k0[s+1] - k0[s]] row-major block of columns [k0[s], k0[s+1]) (equal widths unless the
// plan was given its own); piece s*shards + j is slice s of shard j (rows [j*rows_per_shard,
// (j+1)*rows_per_shard)). A workgroup owns one tile of C for all of K, keeps its accumulators in
// registers, and before each slice waits for the pieces that cover its rows.
struct Resident2DLaunch {
    GemmLaunch g;                 // A = K-sliced base, Wt, C, ldc, N, K (whole), gate; other fields unused
    int32_t M, slices, shards, rows_per_shard;
    const int32_t *k0;            // device, slices + 1 entries: first column of each slice, then K (multiples of the k-tile)
    uint32_t *ticket;
    uint32_t ticket_base[8];
    int32_t grid;
    HandOut out;
    int32_t gated;                // 0: operands resident, no waiting
    int32_t group, col_lists;     // tile order, as in ResidentLaunch
    RunExit leave;
};

// One receiver-side reduction (see ficco_reduce.hip): `in` is the landing buffer [G][rows][N] of the
// peers' partial blocks (slot `block` is not read), `own` this GPU's own partial block, `out` the
// reduced block; a block is `pieces` pieces of piece_vecs 16-byte vectors each; piece s of peer p is
// gate piece p * pieces + s.
struct ReduceLaunch {
    const uint16_t *in;
    const uint16_t *own;
    uint16_t *out;
    int64_t piece_vecs;
    int32_t G, block, pieces, gated;
    Gate gate;
};
hipError_t launch_reduce(const ReduceLaunch &r, int grid, hipStream_t s);
int reduce_grid_size(int device);

// Grouped (per-expert) resident GEMM over ragged row segments. row_tiles: n_row_tiles entries of
// kRowTileWords int32 {first row, rows (1..BM), expert, first piece, last piece, 0, 0, 0} in the order
// they become ready; a tile waits for pieces first..last (ids into the gate's tables) and multiplies
// its rows by Wt + expert * N * K.
constexpr int kRowTileWords = 8;
struct GroupedLaunch {
    GemmLaunch g;                 // A, Wt (all experts, [E][N][K]), C, lda, ldc, N, K, gate
    const int32_t *row_tiles;
    int32_t n_row_tiles;
    uint32_t *ticket;
    uint32_t ticket_base[8];
    int32_t grid;
    HandOut out;
    int32_t gated;
    int32_t group, col_lists;     // tile order, as in ResidentLaunch
};
hipError_t launch_grouped(int tile, const GroupedLaunch &a, hipStream_t s);
int grouped_grid_size(int tile, int device);

hipError_t launch_gemm(int tile, const GemmLaunch &a, hipStream_t s);
hipError_t launch_resident2d(int tile, const Resident2DLaunch &a, hipStream_t s);
int resident2d_grid_size(int tile, int device);
hipError_t launch_resident(int tile, const ResidentLaunch &a, hipStream_t s);
// One wavefront that waits (bounded) until the pieces chunks[0..n) are ready; used to join the
// compute stream with copy-engine transfers when no GEMM consumes them.
hipError_t launch_wait_ready(const Gate &gate, const int32_t *chunks, int n, hipStream_t s);
// One thread stores 0 into the value word of a completion signal (device-visible address) once everything
// before it on the stream has finished: transfers submitted with that signal as a dependency may start.
hipError_t launch_release_signal(uint64_t value_addr, hipStream_t s);
// Sender-side re-layout for column pieces out of a row-major matrix: piece (slice sl, shard j) = rows
// [j*rows_per_shard, (j+1)*rows_per_shard) x columns [k0[sl], k0[sl+1]) of src [M,K] is written as one
// contiguous block at element M*k0[sl] + j*rows_per_shard*width of dst (the K-sliced layout). Workgroups
// take blocks of rows_per_block rows of a piece, pieces in arrival order; stores go through the caches (a copy
// engine reads them next), and the workgroup that completes a piece (counter never reset: blocks_per_piece
// more per run) stores 0 into the value word of that piece's signal, which lets its transfer go.
struct SliceLaunch {
    const uint16_t *src;
    uint16_t *dst;
    int64_t M, K;
    int32_t shards, rows_per_shard;
    const int32_t *k0;            // device, slices + 1 entries
    const int32_t *arrival;       // device, piece ids (sl*shards + j) in arrival order
    int32_t n_pieces, rows_per_block, blocks_per_piece;
    uint32_t *done_count;         // device, per piece id
    const uint64_t *done_sig;     // device, per piece id: address of the signal's value word
};
hipError_t launch_slice_source(const SliceLaunch &a, hipStream_t s);
// C = A * W with W row-major, in one launch of tiles of 16 * row_blocks (1, 2 or 4) rows x 64 columns. W 16-byte aligned,
// C must not overlap W (it is read until the end).
struct DirectLaunch {
    const uint16_t *A, *W;
    uint16_t *C;
    int32_t M, N, K;
    int32_t tiles_m, tiles_n;     // set by the launcher
};
hipError_t launch_direct(int row_blocks, const DirectLaunch &a, hipStream_t s);
// W[K,N] -> Wt[N,K]; also clears up to 256 words at `clear`
hipError_t launch_pack_weight(const uint16_t *W, uint16_t *Wt, int64_t K, int64_t N, hipStream_t s, uint32_t *clear = nullptr, int clear_words = 0);
int resident_grid_size(int tile, int device);

}  // namespace ficco
