// Work lists of the pair kernels: how an ensemble's all-pairs sum (Sec.
// II.C, Eq. superposition) is cut into blocks of (target tile, source chunk)
// and in which order the blocks are dispatched.  Host code only; the order
// and the cut change no result beyond the rounding of the split-K sum, which
// is fixed for a given configuration.
#include <algorithm>
#include <climits>
#include <vector>

#include "mrs_runtime.h"

namespace mrs {

// Default pair-kernel configuration for an ensemble of N points.  Small
// ensembles (split_mode) use the wave-split kernel; larger ones the
// LDS-tiled kernel with 1 (FP32C) or 2 (FP64; 1 for mid-size grids, below)
// targets per lane and
// enough source chunks that the grid holds ~64 blocks per compute unit
// (short blocks keep the tail of the grid short; measured on MI355X at
// 12,800 and 256,000 points).  A chunk has at least 128 sources (64 in small
// grids) and at least N/64, so the split-K partials stay a small fraction of
// the pair work.
//
// Tail split (automatic FP32C tiled configurations of grids of at least four
// blocks per compute unit): the last ~8% of the sources of every target tile
// go into chunks of a quarter chunk (at least 64 sources) whose blocks are
// dispatched last.  A SIMD issues the oldest of its waves first, so the waves
// that start last run alone at the end of the grid; short ones keep that end
// short (measured on MI355X: pair kernel -3.4% at 12,800 points, -0.6% at
// 256,000).  The FP64 kernel (two targets per lane, three resident blocks per CU)
// keeps equal chunks: with the tail split 12,800 points take 314.6 instead of
// 298.7 us, 19,200 points 670 instead of 655; on the persistent schedule it gains
// from about 25,600 points on (1,160 -> 1,126 us; 51,200 points 4,464 -> 4,424,
// of which the longer reduction takes 4 back).
constexpr int kTailPercent = 8, kTailDiv = 4;

// Blocks of the tiled kernel at `tpl` targets per lane and 128-source chunks.
static int64_t blocks_at(int64_t N, int tpl) {
    const int64_t tiles = (N + (int64_t)kBlock * tpl - 1) / ((int64_t)kBlock * tpl);
    return tiles * ((N + 2 * kKahanBlock - 1) / (2 * kKahanBlock));
}

// Mid-size and small grids (measured on MI355X, interleaved A/B against the
// previous rule).  The FP64 kernel takes one target per lane when two would
// give fewer than three blocks per compute unit: twice the waves hide the
// FP64 latency of the near-pair and contact work (3,200 to 6,400 points:
// -7% to -17% alone, -1% to -2% in batches of 16; neutral at 7,680).  When
// 128-source chunks give at most one block per compute unit, chunks shrink
// to 64 sources (2,048 points FP32C: -26% alone, neutral batched; 1,275
// points, 25 swimmers: FP64 23 -> 15 us, and FP32C 48 -> 31 us before that
// size moved to the wave-split kernel).
static bool fp64_one_target(int64_t N, int n_cu) { return blocks_at(N, 2) < (int64_t)3 * n_cu; }
static bool small_grid(int64_t N, int tpl, int n_cu) { return blocks_at(N, tpl) <= (int64_t)n_cu; }

// Ensembles up to 1,024 points use the wave-split kernel (one target per
// wave, lanes split the sources), in both precisions.  In FP32C it is much
// faster alone and loses in deep batches (MI355X, pair + reduction kernels,
// wave-split and tiled, alone, in batches of 4 and of 16: 512 points 10.4 and
// 20.3, 12.2 and 21.2, 22.0 and 21.9 us; 768 points 12.3 and 21.3, 15.3 and 21.4,
// 33.4 and 26.9; 1,024 points 13.5 and 20.9, 20.6 and 21.6, 52.1 and 34.2; 1,280
// points 16.1 and 21.0, 26.6 and 22.1, 73.5 and 44.3): the line lies where
// batches of 4 still gain.  In FP64 the tiled kernel, in quarters of its items,
// is as fast alone from 768 points on and the faster one in batches (512 points
// 11.4 and 12.2, 12.2 and 11.8, 21.9 and 18.4 us; 768 points 11.8 and 11.5, 15.9
// and 15.3, 34.4 and 28.9; 1,024 points 13.2 and 12.0, 21.6 and 18.9, 54.1 and
// 44.8); the line dates from before the quarters.
static bool split_mode(int64_t N, int) { return N <= 1024; }

// Automatic tiled configurations with at least this many blocks per CU run
// the persistent schedule (blocks claim items from a queue).  FP32C, five
// blocks per CU resident (pair + reduction kernels, grid and persistent): 19,200
// points (20 blocks per CU) 335 and 361 us, 25,600 (27) 568 and 591, 38,400 (41)
// 1,242 and 1,239, 51,200 (57) 2,176 and 2,150, 89,600 (91) 6,603 and 6,475.  FP64
// at two targets per lane, three resident (pair kernel): 12,800 points (5) 298
// and 308 us, 19,200 (9) 656 and 660, 25,600 (11) 1,198 and 1,162, 38,400 (18)
// 2,578 and 2,535, 51,200 (24) 4,548 and 4,489, 64,000 (31) 7,102 and 6,994
// (MI355X).  So FP32C crosses at about 40 blocks per CU, close to the line, and
// FP64 at about 10: its line was drawn when four blocks of it were resident.
constexpr int kPersistentBlocksPerCu = 48, kPersistentBlocksPerCuF64T2 = 24;

PairCfg choose_cfg_for(const PairCfg *tuned, int64_t N, int prec, int n_cu) {
    PairCfg c;
    bool small = false;
    if (tuned) {
        c = *tuned;
        if (c.mode == PAIR_QUAD && prec != MRS_FP32C) c.mode = PAIR_TILE;  // the four-wave split is FP32C only
        if (c.mode == PAIR_QUAD) c.tpl = 1;
    } else {
        c.mode = split_mode(N, prec) ? PAIR_SPLIT : PAIR_TILE;
        c.tpl = (prec == MRS_FP32C) ? 1 : 2;
        c.K = 0;
        if (c.mode == PAIR_TILE && prec == MRS_FP64 && fp64_one_target(N, n_cu)) c.tpl = 1;
    }
    // automatic chunking (also of a stored configuration with chunks = 0):
    // 64-source chunks in small grids, as without a stored configuration
    if (c.mode == PAIR_TILE && c.K <= 0) small = small_grid(N, c.tpl, n_cu);
    if (c.mode == PAIR_SPLIT) {
        c.K = 1;
        c.chunk = (int)N;
        return c;
    }
    const int64_t tile = c.mode == PAIR_QUAD ? 64 : (int64_t)kBlock * c.tpl;
    const int64_t tiles = (N + tile - 1) / tile;
    int64_t chunk;
    const bool automatic = c.K <= 0;
    if (automatic) {
        const int64_t want_blocks = (int64_t)n_cu * 64;
        const int64_t K = (want_blocks + tiles - 1) / tiles;
        chunk = std::max<int64_t>({(N + K - 1) / K, (int64_t)(small ? 1 : 2) * kKahanBlock, N / 64});
    } else {
        chunk = (N + c.K - 1) / c.K;
    }
    chunk = ((chunk + kKahanBlock - 1) / kKahanBlock) * kKahanBlock;
    c.chunk = (int)std::max<int64_t>(chunk, kKahanBlock);
    c.K = (int)std::max<int64_t>(1, (N + c.chunk - 1) / c.chunk);
    c.k_big = c.K;
    c.tail_start = c.tail_chunk = 0;
    const int64_t deep = prec == MRS_FP64 && c.tpl == 2 ? kPersistentBlocksPerCuF64T2 : kPersistentBlocksPerCu;
    if (!tuned && c.mode == PAIR_TILE && tiles * c.K >= deep * n_cu) c.sched = SCHED_PERSISTENT;
    if (automatic && prec == MRS_FP32C && tiles * c.K >= (int64_t)4 * n_cu) {
        const int64_t tc = std::max<int64_t>(kKahanBlock, (c.chunk / kTailDiv + kKahanBlock - 1) / kKahanBlock * kKahanBlock);
        const int64_t tail = (N * kTailPercent / 100 + tc - 1) / tc * tc;
        const int64_t B = (N - tail) / kKahanBlock * kKahanBlock;
        if (B > c.chunk) {
            c.tail_start = (int)B;
            c.tail_chunk = (int)tc;
            c.k_big = (int)((B + c.chunk - 1) / c.chunk);
            c.K = c.k_big + (int)((N - B + tc - 1) / tc);
        }
    }
    return c;
}

// FP32C ensembles that the FP64 kernels sum faster (with REC_WIDE records, so
// no value loses precision).  Wave-split configurations always: the launch is
// bound by latency and its near pairs are FP64 anyway (whole evaluations, FP32C
// records and these, alone and in batches of 256: 128 points 21.7 -> 19.7 and
// 85.7 -> 77.0 us; 512 points 23.8 -> 22.0 and 318.6 -> 245.0; 1,024 points 27.3 ->
// 25.0 and 828 -> 734; 20 swimmers in contact, 1,020 points, 44.3 -> 27.3 and in
// batches of 128 691 -> 415).  One target per lane with contact forces up to
// kWideContactPoints: the FP32 kernel sums every contact source in FP64 for every
// target after its own pass, a chain that a small grid waits for.  Deep batches
// fill the chip with either kernel and run at their rates, FP32C's the higher one
// (whole evaluations, FP32C records and these, alone and in batches of 4, 8, 16
// and 32: 1,275 points 56 -> 29, 64 -> 41, 73 -> 55, 103 -> 88, 154 -> 155; 1,785
// points 63 -> 34, 73 -> 55, 94 -> 87, 135 -> 149, 221 -> 272; 2,550 points 67 ->
// 43, 92 -> 84, 131 -> 146, 210 -> 269, 372 -> 513; 3,162 points 81 -> 51, 110 ->
// 115, 171 -> 204, 284 -> 386, 509 -> 747).  An ensemble has to give the same bits
// alone and in a batch, so one rule serves both: the line lies where an ensemble
// alone, the ordinary call, still gains a third, and batches of eight and more of
// the larger ones pay for it.  Without contact forces the FP32C kernel wins in
// batches (1,152 points: 22 us against 29).
constexpr int64_t kWideContactPoints = 3200;

bool wide_records(const PairCfg &c, int64_t N, int prec, bool has_lj) {
    if (prec != MRS_FP32C) return false;
    return c.mode == PAIR_SPLIT || (c.mode == PAIR_TILE && c.tpl == 1 && has_lj && N <= kWideContactPoints);
}

// Ensembles whose FP64 sum at one target per lane runs in quarters of the work
// items (k_pairs_tile_f64).  Alone that fills the chip better; in deep batches its
// block sums, taken four times as often, cost 2 to 6% (whole evaluations, whole
// items and quarters, alone and in batches of 4, 8, 16 and 32: 1,080 points 31.0 ->
// 25.3, 40.1 -> 34.5, 50 -> 46, 77 -> 73, 120 -> 120 us; 1,500 points 32.2 -> 28.2,
// 49 -> 44, 70 -> 65, 106 -> 107, 183 -> 191; 2,048 points 32.9 -> 30.3, 60 -> 59, 94
// -> 96, 160 -> 168, 292 -> 313; 2,500 points 41.5 -> 38.3, 86 -> 82, 136 -> 138, 239
// -> 250, 451 -> 479; 3,200 points 56 -> 46, 121 -> 112, 202 -> 198, 366 -> 372, 692 ->
// 717; pair kernel alone at 3,968 points 39.9 -> 36.0 but in batches of eight 247 ->
// 252, at 5,120 68 -> 59 but 395 -> 415; MI355X).  As above one rule serves both;
// the line lies where batches of eight lose 2% at most.
constexpr int64_t kQuarterPoints = 3200;

void add_items(Plan &P, int e, int64_t N, int n_fil, const PairCfg &c) {
    if (c.mode != PAIR_SPLIT && c.sched == SCHED_PERSISTENT) P.sched = SCHED_PERSISTENT;
    if (c.mode == PAIR_SPLIT) {
        for (int64_t t0 = 0; t0 < N; t0 += kSplitTargetsPerBlock)
            P.split.push_back({e, (int)t0, (int)std::min<int64_t>(kSplitTargetsPerBlock, N - t0), 0, (int)N, 0});
    } else {
        const bool quad = c.mode == PAIR_QUAD;
        const int64_t tile = quad ? 64 : (int64_t)kBlock * c.tpl;
        const bool quart = !quad && c.tpl == 1 && (c.wide || (P.prec == MRS_FP64 && N <= kQuarterPoints));
        auto &dst = quad ? P.quad : (quart ? P.quart : (c.tpl == 2 ? P.tile2 : P.tile1));
        auto &tail = quad ? P.tailq : (quart ? P.tailr : (c.tpl == 2 ? P.tail2 : P.tail1));
        // chunk-major: consecutive blocks share a source chunk, so every XCD
        // (blocks go to the 8 XCDs in turn) reads each chunk once into its L2
        const int64_t B = c.tail_start > 0 ? c.tail_start : N;  // end of the regular chunks
        for (int k = 0; k < c.k_big && (int64_t)k * c.chunk < B; k++) {
            const int64_t s0 = (int64_t)k * c.chunk;
            for (int64_t t0 = 0; t0 < N; t0 += tile)
                dst.push_back({e, (int)t0, (int)std::min<int64_t>(tile, N - t0), (int)s0,
                               (int)std::min<int64_t>(c.chunk, B - s0), k});
        }
        int k = c.k_big;
        for (int64_t s0 = B; s0 < N; s0 += c.tail_chunk, k++)
            for (int64_t t0 = 0; t0 < N; t0 += tile)
                tail.push_back({e, (int)t0, (int)std::min<int64_t>(tile, N - t0), (int)s0,
                                (int)std::min<int64_t>(c.tail_chunk, N - s0), k});
    }
    for (int f = 0; f < n_fil; f++) P.rods.push_back({e, f});
    // the tiled kernels read the source-block descriptors, which the rod
    // launch writes: one item per kBlock / 64 blocks
    if (c.mode != PAIR_SPLIT && n_fil > 0) {
        const int64_t groups = (N + kBlock - 1) / kBlock;
        for (int64_t g = 0; g < groups; g++) P.rods.push_back({e, (int)(-1 - g)});
    }
    for (int64_t p0 = 0; p0 < N; p0 += kReducePoints) P.pts.push_back({e, (int)p0});
    P.pairs_per_eval += N * N;
}

// Blocks whose source range overlaps their own targets in index order hold
// the near pairs along each filament (masked path plus the FP64 rescan) and
// run longest; dispatching them first keeps them off the tail of a launch.
// The order of blocks does not change any result: each writes its own slots.
void near_blocks_first(std::vector<PairItem> &v) {
    std::stable_partition(v.begin(), v.end(), [](const PairItem &it) {
        return it.src0 < it.tgt0 + it.ntgt + kKahanBlock && it.tgt0 < it.src0 + it.nsrc + kKahanBlock;
    });
}

void order_items(Plan &P) {
    near_blocks_first(P.tile1);
    near_blocks_first(P.tile2);
    near_blocks_first(P.quad);
    near_blocks_first(P.quart);
    P.tile1.insert(P.tile1.end(), P.tail1.begin(), P.tail1.end());
    P.tile2.insert(P.tile2.end(), P.tail2.begin(), P.tail2.end());
    P.quad.insert(P.quad.end(), P.tailq.begin(), P.tailq.end());
    P.quart.insert(P.quart.end(), P.tailr.begin(), P.tailr.end());
    P.tail1.clear();
    P.tail2.clear();
    P.tailq.clear();
    P.tailr.clear();
}

// Ensembles of at most kSmallPoints points (the limit's reason: k_small_steps)
// in wave-split configurations, whose sums that kernel repeats; the repulsion
// has passes of its own.
bool small_plan(const Plan &P) {
    for (const EnsDesc &d : P.h_desc)
        if (d.N > kSmallPoints || d.K != 1 || d.has_lj) return false;
    return !P.split.empty() && P.tile1.empty() && P.tile2.empty() && P.quad.empty() && P.quart.empty();
}

}  // namespace mrs

using namespace mrs;

extern "C" mrs_status mrs_plan_items(int64_t n, mrs_precision prec, int32_t n_cu, int32_t *mode,
                                     int32_t *targets_per_lane, int32_t *chunks, int32_t *tail_start,
                                     int32_t *items, int64_t max_items, int64_t *n_items) {
    if (!n_items || n < 1 || n > INT32_MAX / 8 || n_cu < 1 || (prec != MRS_FP64 && prec != MRS_FP32C) ||
        max_items < 0)
        return MRS_EINVAL;
    const PairCfg c = choose_cfg_for(nullptr, n, (int)prec, n_cu);
    Plan P;
    P.prec = (int)prec;
    add_items(P, 0, n, 0, c);
    order_items(P);
    const std::vector<PairItem> &v =
        c.mode == PAIR_SPLIT ? P.split : (c.mode == PAIR_QUAD ? P.quad : (c.tpl == 2 ? P.tile2 : (P.quart.empty() ? P.tile1 : P.quart)));
    *n_items = (int64_t)v.size();
    if (mode) *mode = c.mode;
    if (targets_per_lane) *targets_per_lane = c.tpl;
    if (chunks) *chunks = c.K;
    if (tail_start) *tail_start = c.tail_start > 0 ? c.tail_start : (int32_t)n;
    if (!items) return MRS_OK;
    if (max_items < (int64_t)v.size()) return MRS_EINVAL;
    for (size_t i = 0; i < v.size(); i++) {
        int32_t *o = items + 5 * i;
        o[0] = v[i].tgt0;
        o[1] = v[i].ntgt;
        o[2] = v[i].src0;
        o[3] = v[i].nsrc;
        o[4] = v[i].chunk;
    }
    return MRS_OK;
}
