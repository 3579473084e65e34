// C ABI of libtbik: argument validation, variant choice, launches.  No device memory is allocated here.
#include <algorithm>
#include <atomic>

#include "tbik_internal.hpp"

using namespace tbik;

namespace {

std::atomic<int> g_last_hip_error{0};
std::atomic<int> g_forced_variant{VARIANT_AUTO};

const char *const kVariantNames[VARIANT_COUNT] = {"auto", "reference", "tile128x128", "tile32x128", "tile64x128"};

inline bool is_pow2(int64_t v) { return v >= 1 && (v & (v - 1)) == 0; }
inline bool aligned(const void *p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

int hip_fail(hipError_t e) {
    g_last_hip_error.store((int)e);
    return TBIK_ERR_HIP;
}

// Shape rules common to the GEMM entry points; fills superleaf / ns.
int check_tree(int M, int N, int K, int leaf, int k_first, int P, int *superleaf, int *ns) {
    if (M < 0 || N < 0 || K <= 0 || leaf <= 0 || k_first < 0) return TBIK_ERR_SHAPE;
    if (k_first == 0) {                       // the smallest legal choice: the odd part of the number of leaves
        if (K % leaf != 0) return TBIK_ERR_SHAPE;
        int64_t q = K / leaf;
        while (q % 2 == 0) q /= 2;
        k_first = (int)q;
    }
    const int64_t sl64 = (int64_t)leaf * k_first;
    if (sl64 > K || sl64 % 16 != 0) return TBIK_ERR_SHAPE;
    const int sl = (int)sl64, n = K / sl;
    if (n * sl != K || !is_pow2(n)) return TBIK_ERR_SHAPE;
    if (P < 1 || !is_pow2(P) || P > n || P > TBIK_MAX_SHARDS) return TBIK_ERR_SHARDS;
    *superleaf = sl;
    *ns = n;
    return TBIK_OK;
}

int check_operands(int x_dtype, const void *X, int64_t ldx, const void *W, int64_t ldw, int N, int K) {
    if (!X || !W) return TBIK_ERR_NULL;
    if (ldx < K || ldw < N) return TBIK_ERR_SHAPE;
    const int per16 = (x_dtype == TBIK_F32) ? 4 : 8;       // elements per 16 bytes
    if (!aligned(X, 16) || !aligned(W, 16) || ldx % per16 != 0 || ldw % per16 != 0) return TBIK_ERR_ALIGN;
    return TBIK_OK;
}

// The kernels of an operand format.
bool tiled_supports(const GemmArgs &a, int variant) {
    return a.x_dtype == TBIK_F32 ? gemm_f32_tiled_supports(a) : gemm_tiled_supports(a, variant);
}
hipError_t launch_reference(const GemmArgs &a, hipStream_t s) {
    return a.x_dtype == TBIK_F32 ? launch_gemm_f32_reference(a, s) : launch_gemm_reference(a, s);
}
hipError_t launch_tiled(const GemmArgs &a, int variant, hipStream_t s) {
    return a.x_dtype == TBIK_F32 ? launch_gemm_f32_tiled(a, variant, s) : launch_gemm_tiled(a, variant, s);
}

// Rows of the workgroup tile for a shape (pure): 32 for M <= 32, 64 for M <= 64, else 128 -- unless the 128-row tiles
// would leave a quarter or more of the compute units without one while the 64-row tiles fill exactly one round: then
// 64, which spares the K split (a second launch and an fp32 round trip of the partial sums).  Measured: o_proj
// M = 512 30.6 -> 24.1 us, down_proj M = 512 72.7 -> 61.5 us; with two ragged rounds of 64-row tiles it loses.
int tile_rows(int M, int N) {
    if (M <= 32) return 32;
    if (M <= 64) return 64;
    const int64_t cols = ((int64_t)N + 127) / 128;
    const int64_t tiles128 = (((int64_t)M + 127) / 128) * cols, tiles64 = (((int64_t)M + 63) / 64) * cols;
    return (tiles128 < 192 && tiles64 >= 192 && tiles64 <= 256) ? 64 : 128;
}

// Internal split of K across workgroups (a pure function of the shape, so that tbik_gemm_workspace_bytes() can be
// evaluated without a device): the kernel is launched as if the caller had asked for `split` shards (fp32 partials into
// the workspace) and the partials are combined by the same tree (Theorem 1: identical bits).  Reasons to split: a
// register-resident tree of more than 16 superleaves; fewer than 128 tiles (most compute units idle); and, for very
// long K, rounds -- 256 compute units take the work items in rounds, so 320 tiles cost two rounds of whole-K tiles
// unsplit but five rounds of quarter-K items split in four (32B-class down_proj, K = 25600: M = 1024 454 -> 323 us,
// M = 512 218 -> 189 us, M = 128 78 -> 64 us).  The price of a split is the partials' round trip, the second launch and
// a pipeline fill per item; at K <= 12288 splitting for rounds measured slower (o_proj M = 768: 31 -> 46 us), so this rule
// applies only the first two reasons there (the time model below may still split).
int internal_split(int M, int N, int K, int ns) {
    const int bm = tile_rows(M, N);
    const int64_t tiles = (bm == 32 ? ((int64_t)M + 31) >> 5 : bm == 64 ? ((int64_t)M + 63) >> 6 : ((int64_t)M + 127) >> 7) * (((int64_t)N + 127) / 128);
    int split = 1;
    while (ns > 16 * split && split < TBIK_MAX_SHARDS) split *= 2;   // the tiled kernel walks at most 16 superleaves per shard
    if (K >= 16384) {
        int best = split;
        double best_cost = 0;
        for (int s = split; s <= ns && s <= 16; s *= 2) {
            const double rounds = (double)((tiles * s + 255) / 256);
            const double cost = rounds / s + (s > 1 ? 0.015 + 0.005 * s : 0.0);
            if (s == split || cost < best_cost - 1e-9) { best = s; best_cost = cost; }
        }
        return best;
    }
    if (tiles >= 128) return split;             // at least half of the 256 compute units already have a tile
    while (split < ns && split < 16 && tiles * split < 256) split *= 2;
    return split;
}

// Tile height and K split of a shape for 16-bit and 8-bit operands (pure, given the room for planes), by a model of the time:
//   rounds x max(stages x step[height] + fill, weight bytes of an item / intake) + (split ? combine + planes / rate : 0)
// with rounds = work items / 256 compute units, rounded up.  What the two rules above miss is how evenly the items fill the
// compute units and that a lower tile is cheaper than a padded one: 100 rows of 4096 x 4096 in 8-bit operands took 128-row
// tiles split in eight, 18.2 us from HBM and 15.0 from the cache, and take 14.5 and 10.9 us as unsplit 32-row tiles; 400 rows at K =
// 12288 in bf16 took 224 tiles of 64 rows, 85 us, and take 61 us as 128-row tiles split in two.  The constants were fitted to measured times; they are not
// physical rates one by one (the same planes move at 12 TB/s in one row and at 1.2 in another), and the time they give is
// off by -44 .. +33 % for 16-bit operands, -50 .. +20 % for the others: they rank plans, no more.  Checked over 292 (16-bit)
// and 4 x 99 (low-bit) shapes of the tests' layers, 1 .. 4096 rows, each timed at every height and split, with weights from
// HBM and with weights from the memory-side cache (profiles/tile_split_plans.csv).  The chosen plan, cuts included, takes of
// the rules' time, from HBM / from the cache in the geometric mean: 0.918 / 0.926 (16-bit), 0.935 / 0.904 (8-bit), 0.973 / 0.932
// (MXFP8), 0.941 / 0.902 (MXFP4), 0.955 / 0.947 (MXFP6); from the cache nowhere more than 1.04, from HBM up to 1.09, but 1.21 for 77
// rows of 4096 x 6144 in MXFP8 (32-row tiles unsplit 24.0 us against 19.9, from the cache 13.1 against 18.8) and 1.16 for 64 rows of
// 4096 x 4096 in MXFP4.  Of the best plan's in one piece it takes 0.996 .. 1.014 in the mean, up to 1.22, 1.43 for those 77 rows (the
// epilogue of ragged tiles has become quicker since the constants were fitted, most of all for plans of many 128-row items).  The
// rules' choice stays where the model promises less than the margin.  A tile of 64 rows that the model took too cheap was split
// where the rule is quicker by a tenth (768 rows of 4096 x 6144 from HBM 79 against 71 us, 64 now, cut behind 640).
// 65 .. 96 rows of 16-bit operands may also be one tile of 96 rows, which multiplies a quarter less padding than one of 128 and
// is split like it.  From HBM / from the cache, 77 rows: 4096 x 6144 22.7 -> 19.2 / 17.4 -> 15.8 us, K = 12288 36.1 -> 31.3 /
// 25.4 -> 24.7, 5120 x 7168 27.0 -> 23.6 / 20.3 -> 19.5; 65 rows at K = 14336 39.1 -> 32.8 / 27.2 -> 26.7.  Over 78 shapes of 65 .. 96 rows
// (13 layers; HBM and cache together) its step of 0.46 gives 0.934 of the time without it, nowhere more than 1, and 1.001 of the best plan's;
// 0.42 also takes 2048 x 4096, which loses 8 %, and 0.48 gives 0.950.  More than one tile of 96 was not measured and is not offered.
enum Operands { OPERANDS_16BIT, OPERANDS_FP8, OPERANDS_MXFP8, OPERANDS_MXFP4, OPERANDS_MXFP6 };
struct TilePlan {
    int rows, split;
};
struct TileModel {
    int stage_k;                        // k of an LDS stage
    double bytes_per_k;
    double step[4], fill;               // us: a stage of a 32-, 64-, 96- (16-bit only), 128-row tile; pipeline fill and epilogue of an item
    double intake;                      // bytes of W per us and compute unit, in thousands
    double combine, rate;               // us; bytes of planes per us, in millions
    double retile;                      // us: the scales' re-tiling from 128 rows on
    double margin;                      // the rules' choice stays where the model promises less than this
    double cut;                         // us: a batch stays whole where the model promises less than this from a cut (below)
};
constexpr TileModel kTileModels[] = {
    {64, 2.0, {0.005, 0.25, 0.46, 0.525}, 5.9, 38.5, 3.95, 12.0, 0.0, 1.04, 0.0},
    {128, 1.0, {0.01, 0.24, 0.0, 0.33}, 3.1, 51.0, 2.7, 1.2, 0.0, 1.04, 1.375},
    {128, 1.0, {0.0, 0.185, 0.0, 0.356}, 3.6, 42.0, 4.8, 2.5, 4.0, 1.08, 1.4},
    {256, 0.5, {0.325, 0.335, 0.0, 0.574}, 4.1, 31.4, 2.64, 2.7, 4.0, 1.04, 1.9},
    {128, 0.75, {0.0, 0.0, 0.0, 0.61}, 3.6, 36.0, 3.84, 2.5, 4.0, 1.0, 1.9},       // one height; MXFP8's with its stage
};

// Bytes of the fp32 planes of a K split.
inline size_t split_planes_bytes(int M, int N, int split) { return split > 1 ? (size_t)split * (size_t)M * (size_t)N * sizeof(float) : 0; }

// The model's time of a shape's plans.  The plan is chosen on every call, so what does not depend on it is worked out once
// (a split is a power of two: scaling by it is exact) and rounds are counted in integers.
struct PlanTimes {
    const TileModel &m;
    int64_t M, cols;
    double stages, weights_us, planes_us, retile_us;    // of one shard
    PlanTimes(const TileModel &model, int rows_in_all, int N, int K)
        : m(model), M(rows_in_all), cols(((int64_t)N + 127) / 128), stages((double)K / m.stage_k),
          weights_us(128.0 * K * m.bytes_per_k / (m.intake * 1e3)), planes_us((double)M * N * 4.0 / (m.rate * 1e6)),
          retile_us(M >= 128 ? m.retile : 0.0) {}
    int64_t row_tiles(int rows) const { return rows == 32 ? (M + 31) >> 5 : rows == 64 ? (M + 63) >> 6 : rows == 96 ? (M + 95) / 96 : (M + 127) >> 7; }
    double us(int64_t tiles, double step, int split, double per_split) const {      // per_split: 1 / split
        const double rounds = (double)((tiles * split + 255) >> 8);
        const double item = std::max(stages * per_split * step + m.fill, weights_us * per_split);
        return retile_us + rounds * item + (split > 1 ? m.combine + planes_us * split : 0.0);
    }
    double step(int rows) const { return m.step[rows == 32 ? 0 : rows == 64 ? 1 : rows == 96 ? 2 : 3]; }
    double us(TilePlan p) const { return us(row_tiles(p.rows) * cols, step(p.rows), p.split, 1.0 / p.split); }
};

int forced_rows(int otherwise) {        // what tbik_set_gemm_variant forces
    switch (g_forced_variant.load()) {
        case VARIANT_T128: return 128;
        case VARIANT_T64: return 64;
        case VARIANT_T32: return 32;
        default: return otherwise;
    }
}

// MXFP6 operands have one tile shape (128 x 128), so their rule for the K cut is that of a 128-row tile whatever M.
int mxfp6_split(int M, int N, int ns) {
    const int64_t tiles = (((int64_t)M + 127) / 128) * (((int64_t)N + 127) / 128);
    int split = 1;
    while (ns > 16 * split && split < TBIK_MAX_SHARDS) split *= 2;     // the tiled kernel walks at most 16 superleaves per shard
    if (tiles >= 128) return split;
    while (split < ns && split < 16 && tiles * split < 256) split *= 2;
    return split;
}

struct TimedPlan {
    TilePlan plan;
    double us;
    int rule_split;                     // the older rule's
};
// only_split > 0: the split is the caller's (shard partials), only the height is chosen.  room: bytes for planes.
TimedPlan tile_plan(Operands kind, int M, int N, int K, int ns, int only_split, size_t room) {
    const bool one_height = kind == OPERANDS_MXFP6;
    const TilePlan rule{one_height ? 128 : forced_rows(tile_rows(M, N)),
                        only_split > 0 ? only_split : one_height ? mxfp6_split(M, N, ns) : internal_split(M, N, K, ns)};
    if (g_forced_variant.load() != VARIANT_AUTO || M <= 0 || N <= 0) return {rule, 0.0, rule.split};
    const PlanTimes times(kTileModels[kind], M, N, K);
    const double rule_us = times.us(rule);
    TimedPlan best{rule, rule_us, rule.split};
    double best_us = only_split > 0 || split_planes_bytes(M, N, rule.split) <= room ? rule_us / times.m.margin : 1e30;
    int first_split = only_split > 0 ? only_split : 1;
    while (only_split <= 0 && ns > 16 * (int64_t)first_split) first_split *= 2;         // a tile walks at most 16 superleaves
    const int last_split = only_split <= 0 ? std::min(ns, 16) : only_split <= 16 && ns / only_split <= 16 ? only_split : 0;
    const bool one_tile_of_96 = kind == OPERANDS_16BIT && M > 64 && M <= 96;
    int64_t shorter = 0;
    for (int rows = one_height ? 128 : 32; rows <= 128; rows += rows == 64 && !one_tile_of_96 ? 64 : 32) {
        const int64_t row_tiles = times.row_tiles(rows);
        if (row_tiles == shorter) break;                // a taller tile that does not save one costs more
        shorter = row_tiles;
        const double step = times.step(rows);
        double per_split = 1.0 / first_split;
        for (int split = first_split; split <= last_split; split *= 2, per_split *= 0.5) {
            if (only_split <= 0 && split_planes_bytes(M, N, split) > room) break;
            const double us = times.us(row_tiles * times.cols, step, split, per_split);
            if (us < best_us) { best.plan = {rows, split}; best.us = best_us = us; }
            if ((row_tiles * times.cols * split & 255) == 0) break;       // full rounds: a further split only adds to each
        }
    }
    return best;
}
// Rows of a batch that are better computed by a call of their own (last_rows, 0: none): a launch whose last round of tiles is
// nearly empty is cut behind its last full round, and the remaining rows get the height and split of a small batch.  1100
// rows of 4096 x 4096 in bf16 are 288 tiles of 128 rows, two rounds, 72 us; as 1024 rows and 76 rows 54 us.  (The rows of
// a result do not depend on each other, so neither do their bits.)  Microscaling formats re-tile the scales of both pieces in one
// launch, so a cut pays for it once: at K = 12288 and 1300 rows MXFP8 90.5 -> 82.3 us, MXFP4 59.6 -> 57.0, MXFP6 99.8 -> 95.2.
// A cut that promises less than 5 % or less than the format's `cut` is not made.  Where those lines lie, promised / gained from
// HBM, from the cache, us: 8-bit 1.37 / -1.2, -0.8 (1064 rows at K = 3072), 1.38 / +0.7 .. 4.0, +0.5 .. 2.2 (1152 .. 1280 rows of
// 4096 x 4096, 838 .. 928 at N = 5120; at N = 6144 -0.7, +1.9); MXFP8 1.19 / -2.0, -1.2 (K = 1536), 1.61 / +1.0, +1.5 (K = 3072), 1.78 /
// +4.3, +5.6 (674 rows of 4096 x 6144); MXFP4 1.82 / -0.2, -0.4 (1320 .. 1500 rows), 1.98 / +1.4, +1.7; MXFP6 2.44 /
// +0.4, +1.1 (1029 rows at K = 2048).  For 16-bit operands 5 % is more than 2.1.
constexpr double kPieceUs = 2.0;        // what a launch behind another costs
struct BatchPlan {
    int last_rows;
    TilePlan first, last;               // of the rows before the last ones, of the last ones
    size_t planes, rule_planes;         // bytes that the plans use, that the older rule's split would
};
BatchPlan batch_plan(Operands kind, int M, int N, int K, int ns, size_t room) {
    const TimedPlan whole = tile_plan(kind, M, N, K, ns, 0, room);
    BatchPlan plan{0, whole.plan, whole.plan, split_planes_bytes(M, N, whole.plan.split), split_planes_bytes(M, N, whole.rule_split)};
    if (M <= 0 || N <= 0 || ns > 16 || g_forced_variant.load() != VARIANT_AUTO) return plan;
    const int64_t cols = ((int64_t)N + 127) / 128;
    const int per_round = cols > 256 ? 0 : 256 / (int)cols;                      // row tiles of 128 in a round
    if (per_round < 1 || M <= per_round * 128) return plan;
    const int rest = M % (per_round * 128), full = M - rest;
    if (rest == 0) return plan;
    const TimedPlan first = tile_plan(kind, full, N, K, ns, 0, room), last = tile_plan(kind, rest, N, K, ns, 0, room);
    const double shared_us = rest >= 128 ? kTileModels[kind].retile : 0.0;      // the pieces' scales are re-tiled once
    const double saved_us = whole.us - (first.us + last.us - shared_us + kPieceUs);
    if (saved_us <= 0.05 * whole.us || saved_us < kTileModels[kind].cut) return plan;
    plan.planes = std::max(split_planes_bytes(full, N, first.plan.split), split_planes_bytes(rest, N, last.plan.split));
    plan.last_rows = rest;
    plan.first = first.plan;
    plan.last = last.plan;
    return plan;
}
// The plan of a shape with room for all its planes.  A call asks twice, for the size and for the plan, and a program's layers ask
// for the same few shapes over and over, so a thread remembers what it worked out last (a pure function of the key).  Searching
// each time takes 30 ns in a loop and far more between two launches, where its code and tables are cold: one token 13.0 us, 11.7 so.
const BatchPlan &roomy_plan(Operands kind, int M, int N, int K, int ns) {
    struct Entry {
        int kind, M, N, K, ns;          // ns == 0: empty
        BatchPlan plan;
    };
    constexpr unsigned kEntries = 64;
    static thread_local Entry entries[kEntries];
    Entry &e = entries[((unsigned)M * 7u + ((unsigned)N >> 7) * 13u + ((unsigned)K >> 8) * 29u + (unsigned)ns + (unsigned)kind * 17u) % kEntries];
    if (e.M != M || e.N != N || e.K != K || e.ns != ns || e.kind != (int)kind || g_forced_variant.load() != VARIANT_AUTO) {
        e = {(int)kind, M, N, K, ns, batch_plan(kind, M, N, K, ns, SIZE_MAX)};
        if (g_forced_variant.load() != VARIANT_AUTO) e.ns = 0;     // not remembered
    }
    return e.plan;
}
// Bytes of planes a call can make use of, the older rule's included.
size_t plan_planes_bytes(Operands kind, int M, int N, int K, int ns) {
    const BatchPlan &plan = roomy_plan(kind, M, N, K, ns);
    return std::max(plan.planes, plan.rule_planes);
}
// Calls piece(first row, rows, plan) for the one or two pieces of a batch.
template <class Piece>
hipError_t in_pieces(Operands kind, int M, int N, int K, int ns, size_t room, Piece piece) {
    BatchPlan plan = roomy_plan(kind, M, N, K, ns);
    if (plan.planes > room) plan = batch_plan(kind, M, N, K, ns, room);
    hipError_t e = piece(0, M - plan.last_rows, plan.first);
    return (e == hipSuccess && plan.last_rows > 0) ? piece(M - plan.last_rows, plan.last_rows, plan.last) : e;
}

// fp32 operands: tile height and K split of a shape (pure), by a model of the time.  The fp32 MFMA is slow (a K-step of 32
// takes a 128-row tile 2.0 us and two 32-row tiles side by side on a compute unit 1.05), so what decides is how evenly the work
// items fill 256 compute units: 600 x 2048 at K = 6144 is 80 tiles of 128 rows, which a split in four turns into 320 items = two
// rounds, 198 us; as 304 tiles of 32 rows split in four it is 1216 items, 138 us.  128-row tiles are one per compute unit at a time,
// whole rounds.  32-row tiles are dealt to 512 workgroups, two per compute unit: a last round of up to 256 of them leaves each a
// compute unit to itself and takes 0.93 of 0.62 us a K-step, one of more 1.62 and a full one 1.70.  Checked over 716 shapes (1 .. 1500 rows,
// 512 .. 16384 columns, K = 2048 .. 12288), each timed at every split and both heights: the choice takes 1.004 of the best plan's time in
// the geometric mean, 1.11 at most, and of the older rule's over the 84 of them in profiles/tile_split_plans.csv 0.81, nowhere more.
struct F32Plan {
    int rows, split;
    double us;
};
F32Plan f32_plan_at(int M, int N, int K, int split) {
    const int64_t cols = ((int64_t)N + 127) / 128, items128 = ((int64_t)M + 127) / 128 * cols * split, items32 = ((int64_t)M + 31) / 32 * cols * split;
    const double steps = K / 32.0 / split;
    const double combine = split > 1 ? 4.1 + 0.15 * split + (double)split * M * N * 4.0 / 3e6 : 0.0;
    const int64_t last = items32 & 511;
    const double rounds32 = 1.70 * (double)(items32 >> 9) + (last == 0 ? 0.0 : last <= 256 ? 0.93 : 1.62);
    const double t128 = (double)((items128 + 255) >> 8) * (steps * 2.0 + 1.1) + combine;
    const double t32 = rounds32 * steps * 0.62 + 2.2 + combine;
    return t32 < t128 ? F32Plan{32, split, t32} : F32Plan{128, split, t128};
}
F32Plan f32_plan(int M, int N, int K, int ns) {
    F32Plan best{0, 0, 0.0};
    for (int split = 1; split <= ns && split <= TBIK_MAX_SHARDS; split *= 2) {
        if (ns > 16 * split) continue;                  // the tiled kernel walks at most 16 superleaves per shard
        if (best.rows && split > 16) break;
        const F32Plan p = f32_plan_at(M, N, K, split);
        if (!best.rows || p.us < best.us) best = p;
    }
    if (!best.rows) return F32Plan{128, internal_split(M, N, K, ns), 0.0};
    // Up to 64 rows the older rule's split of 32-row tiles stays where the model promises less than 8 %: 2 rows of 8192 x 8192 split in
    // four take 47.8 us, in eight, held 6 % quicker, 51.3; 64 rows of 4096 x 4096 split in eight 26.9, in four, held 2 % quicker, 28.1.
    // (Above, 128-row tiles were the rule, which leaves the model more to say.)
    if (M <= 64) {
        const F32Plan rule = f32_plan_at(M, N, K, internal_split(M, N, K, ns));
        if (rule.rows == 32 && rule.us < 1.08 * best.us) return rule;
    }
    return best;
}

int pick_variant(const GemmArgs &a, int rows) {      // rows: tile height for 16-bit operands
    const int forced = g_forced_variant.load();
    if (forced != VARIANT_AUTO) return (forced == VARIANT_REFERENCE || tiled_supports(a, forced)) ? forced : VARIANT_REFERENCE;
    if (a.x_dtype == TBIK_F32)
        return !gemm_f32_tiled_supports(a) ? VARIANT_REFERENCE : f32_plan_at(a.M, a.N, a.K, a.P).rows == 32 ? VARIANT_T32 : VARIANT_T128;
    if (rows == 128 && gemm_tiled_supports(a, VARIANT_T128)) return VARIANT_T128;
    if (rows == 96 && gemm_tiled_supports(a, VARIANT_T96)) return VARIANT_T96;
    if (rows >= 64 && gemm_tiled_supports(a, VARIANT_T64)) return VARIANT_T64;
    if (gemm_tiled_supports(a, VARIANT_T32)) return VARIANT_T32;
    if (gemm_tiled_supports(a, VARIANT_T128)) return VARIANT_T128;
    return VARIANT_REFERENCE;
}

// The kernel for a piece of a low-bit call (split: its plan's).  A small batch goes to the one that needs one launch, unless a
// variant is forced.
enum { KERNEL_REFERENCE, KERNEL_TILED, KERNEL_SLICES };
int low_bit_kernel(const GemmArgs &a, const Mxfp4Scales *sc, int split) {
    const int forced = g_forced_variant.load();
    if (forced == VARIANT_AUTO && gemm_slice_takes(a, sc)) return KERNEL_SLICES;
    GemmArgs probe = a;
    probe.P = split;
    const bool tiled = a.x_dtype == TBIK_MXFP4                                   ? gemm_mxfp4_tiled_supports(probe, *sc)
                       : a.x_dtype == TBIK_FP6_E2M3 || a.x_dtype == TBIK_FP6_E3M2 ? gemm_mxfp6_tiled_supports(probe, *sc)
                       : sc                                                       ? gemm_mxfp8_tiled_supports(probe, *sc)
                                                                                  : gemm_fp8_tiled_supports(probe);
    return forced != VARIANT_REFERENCE && tiled ? KERNEL_TILED : KERNEL_REFERENCE;
}

// 16-bit output type that goes with an operand format.
inline bool legal_y_dtype(int y_dtype, int x_dtype) { return y_dtype == TBIK_F32 || y_dtype == x_dtype; }

}  // namespace

extern "C" {

// fp32 partials of the K split, if this shape uses one.
size_t tbik_gemm_16bit_workspace_bytes(int M, int N, int K, int leaf, int k_first) {
    int sl, ns;
    if (check_tree(M, N, K, leaf, k_first, 1, &sl, &ns) != TBIK_OK) return 0;
    return plan_planes_bytes(OPERANDS_16BIT, M, N, K, ns);
}

size_t tbik_gemm_f32_workspace_bytes(int M, int N, int K, int leaf, int k_first) {
    int sl, ns;
    if (check_tree(M, N, K, leaf, k_first, 1, &sl, &ns) != TBIK_OK) return 0;
    return std::max(split_planes_bytes(M, N, internal_split(M, N, K, ns)), split_planes_bytes(M, N, f32_plan(M, N, K, ns).split));
}

size_t tbik_gemm_workspace_bytes(int M, int N, int K, int leaf, int k_first) {
    return std::max(tbik_gemm_16bit_workspace_bytes(M, N, K, leaf, k_first), tbik_gemm_f32_workspace_bytes(M, N, K, leaf, k_first));
}

}  // extern "C"

namespace {

int gemm_shard_partials(int x_dtype, const void *X, int64_t ldx, const void *W, int64_t ldw, float *partials,
                        int M, int N, int K, int leaf, int k_first, int P, void *hip_stream) {
    int sl, ns;
    int rc = check_tree(M, N, K, leaf, k_first, P, &sl, &ns);
    if (rc != TBIK_OK) return rc;
    if (M == 0 || N == 0) return TBIK_OK;
    rc = check_operands(x_dtype, X, ldx, W, ldw, N, K);
    if (rc != TBIK_OK) return rc;
    if (!partials) return TBIK_ERR_NULL;
    if (!aligned(partials, 16)) return TBIK_ERR_ALIGN;
    GemmArgs a{(const uint16_t *)X, ldx, (const uint16_t *)W, ldw, partials, nullptr, 0, TBIK_F32, M, N, K, sl, ns, P, x_dtype};
    hipStream_t s = (hipStream_t)hip_stream;
    const int v = pick_variant(a, tile_plan(OPERANDS_16BIT, M, N, K, ns, P, 0).plan.rows);
    hipError_t e = (v == VARIANT_REFERENCE) ? launch_reference(a, s) : launch_tiled(a, v, s);
    return e == hipSuccess ? TBIK_OK : hip_fail(e);
}

int gemm(int x_dtype, const void *X, int64_t ldx, const void *W, int64_t ldw, void *Y, int64_t ldy,
         int y_dtype, int M, int N, int K, int leaf, int k_first,
         void *workspace, size_t workspace_bytes, void *hip_stream) {
    int sl, ns;
    int rc = check_tree(M, N, K, leaf, k_first, 1, &sl, &ns);
    if (rc != TBIK_OK) return rc;
    if (!legal_y_dtype(y_dtype, x_dtype)) return TBIK_ERR_DTYPE;
    if (M == 0 || N == 0) return TBIK_OK;
    rc = check_operands(x_dtype, X, ldx, W, ldw, N, K);
    if (rc != TBIK_OK) return rc;
    if (!Y) return TBIK_ERR_NULL;
    if (ldy < N) return TBIK_ERR_SHAPE;
    if (!aligned(Y, y_dtype == TBIK_F32 ? 4 : 2)) return TBIK_ERR_ALIGN;
    const size_t need = split_planes_bytes(M, N, internal_split(M, N, K, ns));       // more room may allow a better split
    if (need > 0 && (!workspace || workspace_bytes < need)) return TBIK_ERR_WORKSPACE;
    if (workspace && !aligned(workspace, 256)) return TBIK_ERR_ALIGN;
    const size_t room = workspace ? workspace_bytes : 0;
    hipStream_t s = (hipStream_t)hip_stream;
    auto rows_with = [&](int m0, int m, TilePlan plan) {
        void *y = static_cast<char *>(Y) + (int64_t)m0 * ldy * (y_dtype == TBIK_F32 ? 4 : 2);
        const char *x = static_cast<const char *>(X) + (int64_t)m0 * ldx * (x_dtype == TBIK_F32 ? 4 : 2);
        GemmArgs a{(const uint16_t *)x, ldx, (const uint16_t *)W, ldw, nullptr, y, ldy, y_dtype, m, N, K, sl, ns, 1, x_dtype};
        GemmArgs probe = a;
        probe.P = plan.split;
        const int v = pick_variant(probe, plan.rows);
        if (v == VARIANT_REFERENCE) return launch_reference(a, s);
        if (plan.split == 1) return launch_tiled(a, v, s);
        a.partials = reinterpret_cast<float *>(workspace);
        a.Y = nullptr;
        a.P = plan.split;
        hipError_t e = launch_tiled(a, v, s);
        return e == hipSuccess ? launch_tree_combine(a.partials, plan.split, y, ldy, y_dtype, m, N, s) : e;
    };
    hipError_t e;
    if (x_dtype == TBIK_F32) {                          // its own split, unless the caller brought no room for it
        const int own = f32_plan(M, N, K, ns).split;
        e = rows_with(0, M, {0, own == 1 || split_planes_bytes(M, N, own) <= room ? own : internal_split(M, N, K, ns)});
    } else {
        e = in_pieces(OPERANDS_16BIT, M, N, K, ns, room, rows_with);
    }
    return e == hipSuccess ? TBIK_OK : hip_fail(e);
}

int gemm_reference(int x_dtype, const void *X, int64_t ldx, const void *W, int64_t ldw, float *partials,
                   void *Y, int64_t ldy, int y_dtype,
                   int M, int N, int K, int leaf, int k_first, int P, void *hip_stream) {
    int sl, ns;
    int rc = check_tree(M, N, K, leaf, k_first, P, &sl, &ns);
    if (rc != TBIK_OK) return rc;
    if (!legal_y_dtype(y_dtype, x_dtype)) return TBIK_ERR_DTYPE;
    if (M == 0 || N == 0) return TBIK_OK;
    rc = check_operands(x_dtype, X, ldx, W, ldw, N, K);
    if (rc != TBIK_OK) return rc;
    if (!partials && !Y) return TBIK_ERR_NULL;
    if (Y && P != 1) return TBIK_ERR_SHARDS;
    if (Y && ldy < N) return TBIK_ERR_SHAPE;
    if (Y && !aligned(Y, y_dtype == TBIK_F32 ? 4 : 2)) return TBIK_ERR_ALIGN;
    GemmArgs a{(const uint16_t *)X, ldx, (const uint16_t *)W, ldw, partials, Y, ldy, y_dtype, M, N, K, sl, ns, P, x_dtype};
    hipError_t e = launch_reference(a, (hipStream_t)hip_stream);
    return e == hipSuccess ? TBIK_OK : hip_fail(e);
}

}  // namespace

extern "C" {

int tbik_gemm(const void *X, int64_t ldx, const void *W, int64_t ldw, void *Y, int64_t ldy,
              tbik_dtype y_dtype, int M, int N, int K, int leaf, int k_first,
              void *workspace, size_t workspace_bytes, void *hip_stream) {
    return gemm(TBIK_BF16, X, ldx, W, ldw, Y, ldy, (int)y_dtype, M, N, K, leaf, k_first, workspace, workspace_bytes, hip_stream);
}

int tbik_gemm_f16(const void *X, int64_t ldx, const void *W, int64_t ldw, void *Y, int64_t ldy,
                  tbik_dtype y_dtype, int M, int N, int K, int leaf, int k_first,
                  void *workspace, size_t workspace_bytes, void *hip_stream) {
    return gemm(TBIK_F16, X, ldx, W, ldw, Y, ldy, (int)y_dtype, M, N, K, leaf, k_first, workspace, workspace_bytes, hip_stream);
}

int tbik_gemm_shard_partials(const void *X, int64_t ldx, const void *W, int64_t ldw, float *partials,
                             int M, int N, int K, int leaf, int k_first, int P,
                             void *workspace, size_t workspace_bytes, void *hip_stream) {
    (void)workspace; (void)workspace_bytes;
    return gemm_shard_partials(TBIK_BF16, X, ldx, W, ldw, partials, M, N, K, leaf, k_first, P, hip_stream);
}

int tbik_gemm_shard_partials_f16(const void *X, int64_t ldx, const void *W, int64_t ldw, float *partials,
                                 int M, int N, int K, int leaf, int k_first, int P,
                                 void *workspace, size_t workspace_bytes, void *hip_stream) {
    (void)workspace; (void)workspace_bytes;
    return gemm_shard_partials(TBIK_F16, X, ldx, W, ldw, partials, M, N, K, leaf, k_first, P, hip_stream);
}

int tbik_gemm_reference(const void *X, int64_t ldx, const void *W, int64_t ldw, float *partials,
                        void *Y, int64_t ldy, tbik_dtype y_dtype,
                        int M, int N, int K, int leaf, int k_first, int P, void *hip_stream) {
    return gemm_reference(TBIK_BF16, X, ldx, W, ldw, partials, Y, ldy, (int)y_dtype, M, N, K, leaf, k_first, P, hip_stream);
}

int tbik_gemm_reference_f16(const void *X, int64_t ldx, const void *W, int64_t ldw, float *partials,
                            void *Y, int64_t ldy, tbik_dtype y_dtype,
                            int M, int N, int K, int leaf, int k_first, int P, void *hip_stream) {
    return gemm_reference(TBIK_F16, X, ldx, W, ldw, partials, Y, ldy, (int)y_dtype, M, N, K, leaf, k_first, P, hip_stream);
}

int tbik_gemm_f32(const void *X, int64_t ldx, const void *W, int64_t ldw, void *Y, int64_t ldy,
                  int M, int N, int K, int leaf, int k_first,
                  void *workspace, size_t workspace_bytes, void *hip_stream) {
    return gemm(TBIK_F32, X, ldx, W, ldw, Y, ldy, TBIK_F32, M, N, K, leaf, k_first, workspace, workspace_bytes, hip_stream);
}

int tbik_gemm_shard_partials_f32(const void *X, int64_t ldx, const void *W, int64_t ldw, float *partials,
                                 int M, int N, int K, int leaf, int k_first, int P,
                                 void *workspace, size_t workspace_bytes, void *hip_stream) {
    (void)workspace; (void)workspace_bytes;
    return gemm_shard_partials(TBIK_F32, X, ldx, W, ldw, partials, M, N, K, leaf, k_first, P, hip_stream);
}

int tbik_gemm_reference_f32(const void *X, int64_t ldx, const void *W, int64_t ldw, float *partials,
                            void *Y, int64_t ldy, int M, int N, int K, int leaf, int k_first, int P, void *hip_stream) {
    return gemm_reference(TBIK_F32, X, ldx, W, ldw, partials, Y, ldy, TBIK_F32, M, N, K, leaf, k_first, P, hip_stream);
}

int tbik_tree_combine(const float *partials, int P, void *Y, int64_t ldy, tbik_dtype y_dtype,
                      int M, int N, void *hip_stream) {
    if (M < 0 || N < 0) return TBIK_ERR_SHAPE;
    if (P < 1 || !is_pow2(P) || P > TBIK_MAX_SHARDS) return TBIK_ERR_SHARDS;
    if (y_dtype != TBIK_F32 && y_dtype != TBIK_BF16 && y_dtype != TBIK_F16) return TBIK_ERR_DTYPE;
    if (M == 0 || N == 0) return TBIK_OK;
    if (!partials || !Y) return TBIK_ERR_NULL;
    if (ldy < N) return TBIK_ERR_SHAPE;
    if (!aligned(partials, 16) || !aligned(Y, y_dtype == TBIK_F32 ? 4 : 2)) return TBIK_ERR_ALIGN;
    hipError_t e = launch_tree_combine(partials, P, Y, ldy, (int)y_dtype, M, N, (hipStream_t)hip_stream);
    return e == hipSuccess ? TBIK_OK : hip_fail(e);
}

// ---- 8-bit floating-point operands ----
static bool is_fp8(int d) { return d == TBIK_FP8_E4M3 || d == TBIK_FP8_E5M2; }

static int fp8_checks(int x_dtype, const void *X, int64_t ldx, const void *Wt, int64_t ldwt, int M, int N, int K,
                      int leaf, int k_first, int P, int *sl, int *ns) {
    int rc = check_tree(M, N, K, leaf, k_first, P, sl, ns);
    if (rc != TBIK_OK) return rc;
    if (!is_fp8(x_dtype)) return TBIK_ERR_DTYPE;
    if (*sl % 64 != 0) return TBIK_ERR_SHAPE;
    if (M == 0 || N == 0) return TBIK_OK;
    if (!X || !Wt) return TBIK_ERR_NULL;
    if (ldx < K || ldwt < K) return TBIK_ERR_SHAPE;
    if (!aligned(X, 16) || !aligned(Wt, 16) || ldx % 16 != 0 || ldwt % 16 != 0) return TBIK_ERR_ALIGN;
    return TBIK_OK;
}

size_t tbik_gemm_fp8_workspace_bytes(int M, int N, int K, int leaf, int k_first) {
    int sl, ns;
    if (check_tree(M, N, K, leaf, k_first, 1, &sl, &ns) != TBIK_OK) return 0;
    return plan_planes_bytes(OPERANDS_FP8, M, N, K, ns);
}

int tbik_gemm_fp8(const void *X, int64_t ldx, const void *Wt, int64_t ldwt, void *Y, int64_t ldy,
                  tbik_dtype y_dtype, tbik_dtype x_dtype, int M, int N, int K, int leaf, int k_first,
                  void *workspace, size_t workspace_bytes, void *hip_stream) {
    int sl, ns;
    int rc = fp8_checks((int)x_dtype, X, ldx, Wt, ldwt, M, N, K, leaf, k_first, 1, &sl, &ns);
    if (rc != TBIK_OK) return rc;
    if (y_dtype != TBIK_F32 && y_dtype != TBIK_BF16) return TBIK_ERR_DTYPE;
    if (M == 0 || N == 0) return TBIK_OK;
    if (!Y) return TBIK_ERR_NULL;
    if (ldy < N) return TBIK_ERR_SHAPE;
    if (!aligned(Y, y_dtype == TBIK_F32 ? 4 : 2)) return TBIK_ERR_ALIGN;
    const size_t need = split_planes_bytes(M, N, internal_split(M, N, K, ns));       // more room may allow a better split
    if (need > 0 && (!workspace || workspace_bytes < need)) return TBIK_ERR_WORKSPACE;
    if (workspace && !aligned(workspace, 256)) return TBIK_ERR_ALIGN;
    hipStream_t s = (hipStream_t)hip_stream;
    const size_t room = workspace ? workspace_bytes : 0;
    hipError_t e = in_pieces(OPERANDS_FP8, M, N, K, ns, room, [&](int m0, int m, TilePlan plan) {
        void *y = static_cast<char *>(Y) + (int64_t)m0 * ldy * (y_dtype == TBIK_F32 ? 4 : 2);
        GemmArgs a{(const uint16_t *)(static_cast<const char *>(X) + (int64_t)m0 * ldx), ldx, (const uint16_t *)Wt, ldwt, nullptr, y, ldy,
                   (int)y_dtype, m, N, K, sl, ns, 1, (int)x_dtype, 0};
        const int kernel = low_bit_kernel(a, nullptr, plan.split);
        if (kernel == KERNEL_SLICES) return launch_gemm_slice(a, nullptr, s);
        if (kernel == KERNEL_REFERENCE) return launch_gemm_fp8_reference(a, s);
        if (plan.split == 1) return launch_gemm_fp8_tiled(a, plan.rows, s);
        a.partials = reinterpret_cast<float *>(workspace);
        a.Y = nullptr;
        a.P = plan.split;
        hipError_t pe = launch_gemm_fp8_tiled(a, plan.rows, s);
        return pe == hipSuccess ? launch_tree_combine(a.partials, plan.split, y, ldy, (int)y_dtype, m, N, s) : pe;
    });
    return e == hipSuccess ? TBIK_OK : hip_fail(e);
}

int tbik_gemm_shard_partials_fp8(const void *X, int64_t ldx, const void *Wt, int64_t ldwt, float *partials,
                                 tbik_dtype x_dtype, int M, int N, int K, int leaf, int k_first, int P,
                                 void *workspace, size_t workspace_bytes, void *hip_stream) {
    (void)workspace; (void)workspace_bytes;
    int sl, ns;
    int rc = fp8_checks((int)x_dtype, X, ldx, Wt, ldwt, M, N, K, leaf, k_first, P, &sl, &ns);
    if (rc != TBIK_OK) return rc;
    if (M == 0 || N == 0) return TBIK_OK;
    if (!partials) return TBIK_ERR_NULL;
    if (!aligned(partials, 16)) return TBIK_ERR_ALIGN;
    GemmArgs a{(const uint16_t *)X, ldx, (const uint16_t *)Wt, ldwt, partials, nullptr, 0, TBIK_F32, M, N, K, sl, ns, P, (int)x_dtype, 0};
    const bool tiled = g_forced_variant.load() != VARIANT_REFERENCE && gemm_fp8_tiled_supports(a);
    hipError_t e = tiled ? launch_gemm_fp8_tiled(a, tile_plan(OPERANDS_FP8, M, N, K, ns, P, 0).plan.rows, (hipStream_t)hip_stream)
                         : launch_gemm_fp8_reference(a, (hipStream_t)hip_stream);
    return e == hipSuccess ? TBIK_OK : hip_fail(e);
}

int tbik_gemm_reference_fp8(const void *X, int64_t ldx, const void *Wt, int64_t ldwt, float *partials,
                            void *Y, int64_t ldy, tbik_dtype y_dtype, tbik_dtype x_dtype,
                            int M, int N, int K, int leaf, int k_first, int P, void *hip_stream) {
    int sl, ns;
    int rc = fp8_checks((int)x_dtype, X, ldx, Wt, ldwt, M, N, K, leaf, k_first, P, &sl, &ns);
    if (rc != TBIK_OK) return rc;
    if (y_dtype != TBIK_F32 && y_dtype != TBIK_BF16) return TBIK_ERR_DTYPE;
    if (M == 0 || N == 0) return TBIK_OK;
    if (!partials && !Y) return TBIK_ERR_NULL;
    if (Y && P != 1) return TBIK_ERR_SHARDS;
    if (Y && ldy < N) return TBIK_ERR_SHAPE;
    if (Y && !aligned(Y, y_dtype == TBIK_F32 ? 4 : 2)) return TBIK_ERR_ALIGN;
    GemmArgs a{(const uint16_t *)X, ldx, (const uint16_t *)Wt, ldwt, partials, Y, ldy, (int)y_dtype, M, N, K, sl, ns, P, (int)x_dtype, 0};
    hipError_t e = launch_gemm_fp8_reference(a, (hipStream_t)hip_stream);
    return e == hipSuccess ? TBIK_OK : hip_fail(e);
}

// ---- MXFP4 operands ----
static int mxfp4_checks(const void *X, int64_t ldx, const void *Xs, int64_t ldxs, const void *Wt, int64_t ldwt,
                        const void *Ws, int64_t ldws, int M, int N, int K, int leaf, int k_first, int P, int *sl, int *ns) {
    int rc = check_tree(M, N, K, leaf, k_first, P, sl, ns);
    if (rc != TBIK_OK) return rc;
    if (*sl % 64 != 0) return TBIK_ERR_SHAPE;
    if (M == 0 || N == 0) return TBIK_OK;
    if (!X || !Wt || !Xs || !Ws) return TBIK_ERR_NULL;
    if (ldx < K / 2 || ldwt < K / 2 || ldxs < K / 32 || ldws < K / 32) return TBIK_ERR_SHAPE;
    if (!aligned(X, 16) || !aligned(Wt, 16) || ldx % 16 != 0 || ldwt % 16 != 0) return TBIK_ERR_ALIGN;
    return TBIK_OK;
}

// From 128 rows on the microscaling GEMMs re-tile their scales first (a launch of its own, which a small batch would
// feel): the workspace is the fp32 planes of the K split, rounded up to 256 bytes, then the re-tiled scales.  The pieces of a
// cut batch share one re-tiling.
static bool mx_retiles(int M) { return M >= 128; }
static size_t round_256(size_t bytes) { return (bytes + 255) & ~(size_t)255; }
using RetileScales = hipError_t (*)(const Mxfp4Scales &, int M, int N, int K, void *out, Mxfp4Scales *packed, hipStream_t s);
struct CallScales {
    Mxfp4Scales raw;                    // of the whole call
    int M, N, K;
    RetileScales retile;
    void *area;                         // room for the copies, or nullptr: none are made
    Mxfp4Scales packed{};
    // The scales of the rows from m0 on for the reference kernel and the slices; for the tiled kernels (m0 a multiple of 128).
    Mxfp4Scales plain(int m0) const {
        Mxfp4Scales sc = raw;
        sc.Xs += (int64_t)m0 * raw.ldxs;
        return sc;
    }
    hipError_t for_tiles(int m0, Mxfp4Scales *sc, hipStream_t s) {
        *sc = plain(m0);
        if (!area || (m0 & 127)) return hipSuccess;
        if (!packed.packed) {
            hipError_t e = retile(raw, M, N, K, area, &packed, s);
            if (e != hipSuccess) return e;
        }
        *sc = packed;
        sc->Xs += (int64_t)m0 * (K / 32);
        return hipSuccess;
    }
};
static size_t mxfp4_scales_room(int M, int N, int K) { return mx_retiles(M) && K % 256 == 0 ? mxfp4_retiled_scales_bytes(M, N, K) : 0; }
size_t tbik_gemm_mxfp4_workspace_bytes(int M, int N, int K, int leaf, int k_first) {
    int sl, ns;
    if (check_tree(M, N, K, leaf, k_first, 1, &sl, &ns) != TBIK_OK) return 0;
    return round_256(plan_planes_bytes(OPERANDS_MXFP4, M, N, K, ns)) + mxfp4_scales_room(M, N, K);
}

int tbik_gemm_mxfp4(const void *X, int64_t ldx, const void *Xs, int64_t ldxs, const void *Wt, int64_t ldwt,
                    const void *Ws, int64_t ldws, void *Y, int64_t ldy, tbik_dtype y_dtype,
                    int M, int N, int K, int leaf, int k_first,
                    void *workspace, size_t workspace_bytes, void *hip_stream) {
    int sl, ns;
    int rc = mxfp4_checks(X, ldx, Xs, ldxs, Wt, ldwt, Ws, ldws, M, N, K, leaf, k_first, 1, &sl, &ns);
    if (rc != TBIK_OK) return rc;
    if (y_dtype != TBIK_F32 && y_dtype != TBIK_BF16) return TBIK_ERR_DTYPE;
    if (M == 0 || N == 0) return TBIK_OK;
    if (!Y) return TBIK_ERR_NULL;
    if (ldy < N) return TBIK_ERR_SHAPE;
    if (!aligned(Y, y_dtype == TBIK_F32 ? 4 : 2)) return TBIK_ERR_ALIGN;
    const size_t scales_room = mxfp4_scales_room(M, N, K);
    const size_t need = round_256(split_planes_bytes(M, N, internal_split(M, N, K, ns))) + scales_room;      // more room may allow a better split
    if (need > 0 && (!workspace || workspace_bytes < need)) return TBIK_ERR_WORKSPACE;
    if (workspace && !aligned(workspace, 256)) return TBIK_ERR_ALIGN;
    hipStream_t s = (hipStream_t)hip_stream;
    const size_t room = workspace && workspace_bytes > scales_room ? (workspace_bytes - scales_room) & ~(size_t)255 : 0;      // planes are rounded up to 256 bytes
    CallScales scales{{(const uint8_t *)Xs, ldxs, (const uint8_t *)Ws, ldws}, M, N, K, launch_mxfp4_retile,
                      scales_room ? static_cast<char *>(workspace) + room : nullptr};
    hipError_t e = in_pieces(OPERANDS_MXFP4, M, N, K, ns, room, [&](int m0, int m, TilePlan plan) {
        void *y = static_cast<char *>(Y) + (int64_t)m0 * ldy * (y_dtype == TBIK_F32 ? 4 : 2);
        GemmArgs a{(const uint16_t *)(static_cast<const char *>(X) + (int64_t)m0 * ldx), ldx, (const uint16_t *)Wt, ldwt, nullptr, y, ldy,
                   (int)y_dtype, m, N, K, sl, ns, 1, TBIK_MXFP4, 0};
        const Mxfp4Scales sc = scales.plain(m0);
        const int kernel = low_bit_kernel(a, &sc, plan.split);
        if (kernel == KERNEL_SLICES) return launch_gemm_slice(a, &sc, s);
        if (kernel == KERNEL_REFERENCE) return launch_gemm_mxfp4_reference(a, sc, s);
        Mxfp4Scales tiled;
        hipError_t pe = scales.for_tiles(m0, &tiled, s);
        if (pe != hipSuccess) return pe;
        if (plan.split == 1) return launch_gemm_mxfp4_tiled(a, tiled, plan.rows, s);
        a.partials = reinterpret_cast<float *>(workspace);
        a.Y = nullptr;
        a.P = plan.split;
        pe = launch_gemm_mxfp4_tiled(a, tiled, plan.rows, s);
        return pe == hipSuccess ? launch_tree_combine(a.partials, plan.split, y, ldy, (int)y_dtype, m, N, s) : pe;
    });
    return e == hipSuccess ? TBIK_OK : hip_fail(e);
}

int tbik_gemm_shard_partials_mxfp4(const void *X, int64_t ldx, const void *Xs, int64_t ldxs, const void *Wt, int64_t ldwt,
                                   const void *Ws, int64_t ldws, float *partials,
                                   int M, int N, int K, int leaf, int k_first, int P,
                                   void *workspace, size_t workspace_bytes, void *hip_stream) {
    int sl, ns;
    int rc = mxfp4_checks(X, ldx, Xs, ldxs, Wt, ldwt, Ws, ldws, M, N, K, leaf, k_first, P, &sl, &ns);
    if (rc != TBIK_OK) return rc;
    if (M == 0 || N == 0) return TBIK_OK;
    if (!partials) return TBIK_ERR_NULL;
    if (!aligned(partials, 16)) return TBIK_ERR_ALIGN;
    GemmArgs a{(const uint16_t *)X, ldx, (const uint16_t *)Wt, ldwt, partials, nullptr, 0, TBIK_F32, M, N, K, sl, ns, P, TBIK_MXFP4, 0};
    const Mxfp4Scales sc{(const uint8_t *)Xs, ldxs, (const uint8_t *)Ws, ldws};
    const bool tiled = g_forced_variant.load() != VARIANT_REFERENCE && gemm_mxfp4_tiled_supports(a, sc);
    // a workspace as tbik_gemm_mxfp4 takes it has room for the re-tiled scales
    const bool room = mx_retiles(M) && workspace && aligned(workspace, 256) && workspace_bytes >= mxfp4_scales_room(M, N, K);
    CallScales scales{sc, M, N, K, launch_mxfp4_retile, room ? workspace : nullptr};
    Mxfp4Scales use;
    hipError_t e = tiled ? scales.for_tiles(0, &use, (hipStream_t)hip_stream) : hipSuccess;
    if (e == hipSuccess) e = tiled ? launch_gemm_mxfp4_tiled(a, use, tile_plan(OPERANDS_MXFP4, M, N, K, ns, P, 0).plan.rows, (hipStream_t)hip_stream)
                                   : launch_gemm_mxfp4_reference(a, sc, (hipStream_t)hip_stream);
    return e == hipSuccess ? TBIK_OK : hip_fail(e);
}

int tbik_gemm_reference_mxfp4(const void *X, int64_t ldx, const void *Xs, int64_t ldxs, const void *Wt, int64_t ldwt,
                              const void *Ws, int64_t ldws, float *partials, void *Y, int64_t ldy, tbik_dtype y_dtype,
                              int M, int N, int K, int leaf, int k_first, int P, void *hip_stream) {
    int sl, ns;
    int rc = mxfp4_checks(X, ldx, Xs, ldxs, Wt, ldwt, Ws, ldws, M, N, K, leaf, k_first, P, &sl, &ns);
    if (rc != TBIK_OK) return rc;
    if (y_dtype != TBIK_F32 && y_dtype != TBIK_BF16) return TBIK_ERR_DTYPE;
    if (M == 0 || N == 0) return TBIK_OK;
    if (!partials && !Y) return TBIK_ERR_NULL;
    if (Y && P != 1) return TBIK_ERR_SHARDS;
    if (Y && ldy < N) return TBIK_ERR_SHAPE;
    if (Y && !aligned(Y, y_dtype == TBIK_F32 ? 4 : 2)) return TBIK_ERR_ALIGN;
    GemmArgs a{(const uint16_t *)X, ldx, (const uint16_t *)Wt, ldwt, partials, Y, ldy, (int)y_dtype, M, N, K, sl, ns, P, TBIK_MXFP4, 0};
    const Mxfp4Scales sc{(const uint8_t *)Xs, ldxs, (const uint8_t *)Ws, ldws};
    hipError_t e = launch_gemm_mxfp4_reference(a, sc, (hipStream_t)hip_stream);
    return e == hipSuccess ? TBIK_OK : hip_fail(e);
}

// ---- MXFP8 operands ----
static int mxfp8_checks(int x_dtype, const void *X, int64_t ldx, const void *Xs, int64_t ldxs, const void *Wt, int64_t ldwt,
                        const void *Ws, int64_t ldws, int M, int N, int K, int leaf, int k_first, int P, int *sl, int *ns) {
    int rc = fp8_checks(x_dtype, X, ldx, Wt, ldwt, M, N, K, leaf, k_first, P, sl, ns);
    if (rc != TBIK_OK) return rc;
    if (M == 0 || N == 0) return TBIK_OK;
    if (!Xs || !Ws) return TBIK_ERR_NULL;
    if (ldxs < K / 32 || ldws < K / 32) return TBIK_ERR_SHAPE;
    return TBIK_OK;
}

static size_t mxfp8_scales_room(int M, int N, int K) { return mx_retiles(M) && K % 128 == 0 ? mxfp8_retiled_scales_bytes(M, N, K) : 0; }
size_t tbik_gemm_mxfp8_workspace_bytes(int M, int N, int K, int leaf, int k_first) {
    int sl, ns;
    if (check_tree(M, N, K, leaf, k_first, 1, &sl, &ns) != TBIK_OK) return 0;
    return round_256(plan_planes_bytes(OPERANDS_MXFP8, M, N, K, ns)) + mxfp8_scales_room(M, N, K);
}

int tbik_gemm_mxfp8(const void *X, int64_t ldx, const void *Xs, int64_t ldxs, const void *Wt, int64_t ldwt,
                    const void *Ws, int64_t ldws, void *Y, int64_t ldy, tbik_dtype y_dtype, tbik_dtype x_dtype,
                    int M, int N, int K, int leaf, int k_first,
                    void *workspace, size_t workspace_bytes, void *hip_stream) {
    int sl, ns;
    int rc = mxfp8_checks((int)x_dtype, X, ldx, Xs, ldxs, Wt, ldwt, Ws, ldws, M, N, K, leaf, k_first, 1, &sl, &ns);
    if (rc != TBIK_OK) return rc;
    if (y_dtype != TBIK_F32 && y_dtype != TBIK_BF16) return TBIK_ERR_DTYPE;
    if (M == 0 || N == 0) return TBIK_OK;
    if (!Y) return TBIK_ERR_NULL;
    if (ldy < N) return TBIK_ERR_SHAPE;
    if (!aligned(Y, y_dtype == TBIK_F32 ? 4 : 2)) return TBIK_ERR_ALIGN;
    const size_t scales_room = mxfp8_scales_room(M, N, K);
    const size_t need = round_256(split_planes_bytes(M, N, internal_split(M, N, K, ns))) + scales_room;      // more room may allow a better split
    if (need > 0 && (!workspace || workspace_bytes < need)) return TBIK_ERR_WORKSPACE;
    if (workspace && !aligned(workspace, 256)) return TBIK_ERR_ALIGN;
    hipStream_t s = (hipStream_t)hip_stream;
    const size_t room = workspace && workspace_bytes > scales_room ? (workspace_bytes - scales_room) & ~(size_t)255 : 0;      // planes are rounded up to 256 bytes
    CallScales scales{{(const uint8_t *)Xs, ldxs, (const uint8_t *)Ws, ldws}, M, N, K, launch_mxfp8_retile,
                      scales_room ? static_cast<char *>(workspace) + room : nullptr};
    hipError_t e = in_pieces(OPERANDS_MXFP8, M, N, K, ns, room, [&](int m0, int m, TilePlan plan) {
        void *y = static_cast<char *>(Y) + (int64_t)m0 * ldy * (y_dtype == TBIK_F32 ? 4 : 2);
        GemmArgs a{(const uint16_t *)(static_cast<const char *>(X) + (int64_t)m0 * ldx), ldx, (const uint16_t *)Wt, ldwt, nullptr, y, ldy,
                   (int)y_dtype, m, N, K, sl, ns, 1, (int)x_dtype, 0};
        const Mxfp4Scales sc = scales.plain(m0);
        const int kernel = low_bit_kernel(a, &sc, plan.split);
        if (kernel == KERNEL_SLICES) return launch_gemm_slice(a, &sc, s);
        if (kernel == KERNEL_REFERENCE) return launch_gemm_mxfp8_reference(a, sc, s);
        Mxfp4Scales tiled;
        hipError_t pe = scales.for_tiles(m0, &tiled, s);
        if (pe != hipSuccess) return pe;
        if (plan.split == 1) return launch_gemm_mxfp8_tiled(a, tiled, plan.rows, s);
        a.partials = reinterpret_cast<float *>(workspace);
        a.Y = nullptr;
        a.P = plan.split;
        pe = launch_gemm_mxfp8_tiled(a, tiled, plan.rows, s);
        return pe == hipSuccess ? launch_tree_combine(a.partials, plan.split, y, ldy, (int)y_dtype, m, N, s) : pe;
    });
    return e == hipSuccess ? TBIK_OK : hip_fail(e);
}

int tbik_gemm_shard_partials_mxfp8(const void *X, int64_t ldx, const void *Xs, int64_t ldxs, const void *Wt, int64_t ldwt,
                                   const void *Ws, int64_t ldws, float *partials, tbik_dtype x_dtype,
                                   int M, int N, int K, int leaf, int k_first, int P,
                                   void *workspace, size_t workspace_bytes, void *hip_stream) {
    int sl, ns;
    int rc = mxfp8_checks((int)x_dtype, X, ldx, Xs, ldxs, Wt, ldwt, Ws, ldws, M, N, K, leaf, k_first, P, &sl, &ns);
    if (rc != TBIK_OK) return rc;
    if (M == 0 || N == 0) return TBIK_OK;
    if (!partials) return TBIK_ERR_NULL;
    if (!aligned(partials, 16)) return TBIK_ERR_ALIGN;
    GemmArgs a{(const uint16_t *)X, ldx, (const uint16_t *)Wt, ldwt, partials, nullptr, 0, TBIK_F32, M, N, K, sl, ns, P, (int)x_dtype, 0};
    const Mxfp4Scales sc{(const uint8_t *)Xs, ldxs, (const uint8_t *)Ws, ldws};
    const bool tiled = g_forced_variant.load() != VARIANT_REFERENCE && gemm_mxfp8_tiled_supports(a, sc);
    // a workspace as tbik_gemm_mxfp8 takes it has room for the re-tiled scales
    const bool room = mx_retiles(M) && workspace && aligned(workspace, 256) && workspace_bytes >= mxfp8_scales_room(M, N, K);
    CallScales scales{sc, M, N, K, launch_mxfp8_retile, room ? workspace : nullptr};
    Mxfp4Scales use;
    hipError_t e = tiled ? scales.for_tiles(0, &use, (hipStream_t)hip_stream) : hipSuccess;
    if (e == hipSuccess) e = tiled ? launch_gemm_mxfp8_tiled(a, use, tile_plan(OPERANDS_MXFP8, M, N, K, ns, P, 0).plan.rows, (hipStream_t)hip_stream)
                                   : launch_gemm_mxfp8_reference(a, sc, (hipStream_t)hip_stream);
    return e == hipSuccess ? TBIK_OK : hip_fail(e);
}

int tbik_gemm_reference_mxfp8(const void *X, int64_t ldx, const void *Xs, int64_t ldxs, const void *Wt, int64_t ldwt,
                              const void *Ws, int64_t ldws, float *partials, void *Y, int64_t ldy, tbik_dtype y_dtype,
                              tbik_dtype x_dtype, int M, int N, int K, int leaf, int k_first, int P, void *hip_stream) {
    int sl, ns;
    int rc = mxfp8_checks((int)x_dtype, X, ldx, Xs, ldxs, Wt, ldwt, Ws, ldws, M, N, K, leaf, k_first, P, &sl, &ns);
    if (rc != TBIK_OK) return rc;
    if (y_dtype != TBIK_F32 && y_dtype != TBIK_BF16) return TBIK_ERR_DTYPE;
    if (M == 0 || N == 0) return TBIK_OK;
    if (!partials && !Y) return TBIK_ERR_NULL;
    if (Y && P != 1) return TBIK_ERR_SHARDS;
    if (Y && ldy < N) return TBIK_ERR_SHAPE;
    if (Y && !aligned(Y, y_dtype == TBIK_F32 ? 4 : 2)) return TBIK_ERR_ALIGN;
    GemmArgs a{(const uint16_t *)X, ldx, (const uint16_t *)Wt, ldwt, partials, Y, ldy, (int)y_dtype, M, N, K, sl, ns, P, (int)x_dtype, 0};
    const Mxfp4Scales sc{(const uint8_t *)Xs, ldxs, (const uint8_t *)Ws, ldws};
    hipError_t e = launch_gemm_mxfp8_reference(a, sc, (hipStream_t)hip_stream);
    return e == hipSuccess ? TBIK_OK : hip_fail(e);
}

// ---- MXFP6 operands ----
static int mxfp6_checks(int x_dtype, const void *X, int64_t ldx, const void *Xs, int64_t ldxs, const void *Wt, int64_t ldwt,
                        const void *Ws, int64_t ldws, int M, int N, int K, int leaf, int k_first, int P, int *sl, int *ns) {
    int rc = check_tree(M, N, K, leaf, k_first, P, sl, ns);
    if (rc != TBIK_OK) return rc;
    if (x_dtype != TBIK_FP6_E2M3 && x_dtype != TBIK_FP6_E3M2) return TBIK_ERR_DTYPE;
    if (*sl % 64 != 0) return TBIK_ERR_SHAPE;
    if (M == 0 || N == 0) return TBIK_OK;
    if (!X || !Wt || !Xs || !Ws) return TBIK_ERR_NULL;
    if (ldx < (int64_t)K / 4 * 3 || ldwt < (int64_t)K / 4 * 3 || ldxs < K / 32 || ldws < K / 32) return TBIK_ERR_SHAPE;
    if (!aligned(X, 16) || !aligned(Wt, 16) || ldx % 16 != 0 || ldwt % 16 != 0) return TBIK_ERR_ALIGN;
    return TBIK_OK;
}

static size_t mxfp6_scales_room(int M, int N, int K) { return mx_retiles(M) && K % 128 == 0 ? mxfp6_retiled_scales_bytes(M, N, K) : 0; }
size_t tbik_gemm_mxfp6_workspace_bytes(int M, int N, int K, int leaf, int k_first) {
    int sl, ns;
    if (check_tree(M, N, K, leaf, k_first, 1, &sl, &ns) != TBIK_OK) return 0;
    return round_256(plan_planes_bytes(OPERANDS_MXFP6, M, N, K, ns)) + mxfp6_scales_room(M, N, K);
}

int tbik_gemm_mxfp6(const void *X, int64_t ldx, const void *Xs, int64_t ldxs, const void *Wt, int64_t ldwt,
                    const void *Ws, int64_t ldws, void *Y, int64_t ldy, tbik_dtype y_dtype, tbik_dtype x_dtype,
                    int M, int N, int K, int leaf, int k_first,
                    void *workspace, size_t workspace_bytes, void *hip_stream) {
    int sl, ns;
    int rc = mxfp6_checks((int)x_dtype, X, ldx, Xs, ldxs, Wt, ldwt, Ws, ldws, M, N, K, leaf, k_first, 1, &sl, &ns);
    if (rc != TBIK_OK) return rc;
    if (y_dtype != TBIK_F32 && y_dtype != TBIK_BF16) return TBIK_ERR_DTYPE;
    if (M == 0 || N == 0) return TBIK_OK;
    if (!Y) return TBIK_ERR_NULL;
    if (ldy < N) return TBIK_ERR_SHAPE;
    if (!aligned(Y, y_dtype == TBIK_F32 ? 4 : 2)) return TBIK_ERR_ALIGN;
    const size_t scales_room = mxfp6_scales_room(M, N, K);
    const size_t need = round_256(split_planes_bytes(M, N, mxfp6_split(M, N, ns))) + scales_room;      // more room may allow a better split
    if (need > 0 && (!workspace || workspace_bytes < need)) return TBIK_ERR_WORKSPACE;
    if (workspace && !aligned(workspace, 256)) return TBIK_ERR_ALIGN;
    hipStream_t s = (hipStream_t)hip_stream;
    const size_t room = workspace && workspace_bytes > scales_room ? (workspace_bytes - scales_room) & ~(size_t)255 : 0;      // planes are rounded up to 256 bytes
    CallScales scales{{(const uint8_t *)Xs, ldxs, (const uint8_t *)Ws, ldws}, M, N, K, launch_mxfp6_retile,
                      scales_room ? static_cast<char *>(workspace) + room : nullptr};
    hipError_t e = in_pieces(OPERANDS_MXFP6, M, N, K, ns, room, [&](int m0, int m, TilePlan plan) {
        void *y = static_cast<char *>(Y) + (int64_t)m0 * ldy * (y_dtype == TBIK_F32 ? 4 : 2);
        GemmArgs a{(const uint16_t *)(static_cast<const char *>(X) + (int64_t)m0 * ldx), ldx, (const uint16_t *)Wt, ldwt, nullptr, y, ldy,
                   (int)y_dtype, m, N, K, sl, ns, 1, (int)x_dtype, 0};
        const Mxfp4Scales sc = scales.plain(m0);
        const int kernel = low_bit_kernel(a, &sc, plan.split);
        if (kernel == KERNEL_SLICES) return launch_gemm_slice(a, &sc, s);
        if (kernel == KERNEL_REFERENCE) return launch_gemm_mxfp6_reference(a, sc, s);
        Mxfp4Scales tiled;
        hipError_t pe = scales.for_tiles(m0, &tiled, s);
        if (pe != hipSuccess) return pe;
        if (plan.split == 1) return launch_gemm_mxfp6_tiled(a, tiled, s);
        a.partials = reinterpret_cast<float *>(workspace);
        a.Y = nullptr;
        a.P = plan.split;
        pe = launch_gemm_mxfp6_tiled(a, tiled, s);
        return pe == hipSuccess ? launch_tree_combine(a.partials, plan.split, y, ldy, (int)y_dtype, m, N, s) : pe;
    });
    return e == hipSuccess ? TBIK_OK : hip_fail(e);
}

int tbik_gemm_shard_partials_mxfp6(const void *X, int64_t ldx, const void *Xs, int64_t ldxs, const void *Wt, int64_t ldwt,
                                   const void *Ws, int64_t ldws, float *partials, tbik_dtype x_dtype,
                                   int M, int N, int K, int leaf, int k_first, int P,
                                   void *workspace, size_t workspace_bytes, void *hip_stream) {
    int sl, ns;
    int rc = mxfp6_checks((int)x_dtype, X, ldx, Xs, ldxs, Wt, ldwt, Ws, ldws, M, N, K, leaf, k_first, P, &sl, &ns);
    if (rc != TBIK_OK) return rc;
    if (M == 0 || N == 0) return TBIK_OK;
    if (!partials) return TBIK_ERR_NULL;
    if (!aligned(partials, 16)) return TBIK_ERR_ALIGN;
    GemmArgs a{(const uint16_t *)X, ldx, (const uint16_t *)Wt, ldwt, partials, nullptr, 0, TBIK_F32, M, N, K, sl, ns, P, (int)x_dtype, 0};
    const Mxfp4Scales sc{(const uint8_t *)Xs, ldxs, (const uint8_t *)Ws, ldws};
    const bool tiled = g_forced_variant.load() != VARIANT_REFERENCE && gemm_mxfp6_tiled_supports(a, sc);
    // a workspace as tbik_gemm_mxfp6 takes it has room for the re-tiled scales
    const bool room = mx_retiles(M) && workspace && aligned(workspace, 256) && workspace_bytes >= mxfp6_scales_room(M, N, K);
    CallScales scales{sc, M, N, K, launch_mxfp6_retile, room ? workspace : nullptr};
    Mxfp4Scales use;
    hipError_t e = tiled ? scales.for_tiles(0, &use, (hipStream_t)hip_stream) : hipSuccess;
    if (e == hipSuccess) e = tiled ? launch_gemm_mxfp6_tiled(a, use, (hipStream_t)hip_stream)
                                   : launch_gemm_mxfp6_reference(a, sc, (hipStream_t)hip_stream);
    return e == hipSuccess ? TBIK_OK : hip_fail(e);
}

int tbik_gemm_reference_mxfp6(const void *X, int64_t ldx, const void *Xs, int64_t ldxs, const void *Wt, int64_t ldwt,
                              const void *Ws, int64_t ldws, float *partials, void *Y, int64_t ldy, tbik_dtype y_dtype,
                              tbik_dtype x_dtype, int M, int N, int K, int leaf, int k_first, int P, void *hip_stream) {
    int sl, ns;
    int rc = mxfp6_checks((int)x_dtype, X, ldx, Xs, ldxs, Wt, ldwt, Ws, ldws, M, N, K, leaf, k_first, P, &sl, &ns);
    if (rc != TBIK_OK) return rc;
    if (y_dtype != TBIK_F32 && y_dtype != TBIK_BF16) return TBIK_ERR_DTYPE;
    if (M == 0 || N == 0) return TBIK_OK;
    if (!partials && !Y) return TBIK_ERR_NULL;
    if (Y && P != 1) return TBIK_ERR_SHARDS;
    if (Y && ldy < N) return TBIK_ERR_SHAPE;
    if (Y && !aligned(Y, y_dtype == TBIK_F32 ? 4 : 2)) return TBIK_ERR_ALIGN;
    GemmArgs a{(const uint16_t *)X, ldx, (const uint16_t *)Wt, ldwt, partials, Y, ldy, (int)y_dtype, M, N, K, sl, ns, P, (int)x_dtype, 0};
    const Mxfp4Scales sc{(const uint8_t *)Xs, ldxs, (const uint8_t *)Ws, ldws};
    hipError_t e = launch_gemm_mxfp6_reference(a, sc, (hipStream_t)hip_stream);
    return e == hipSuccess ? TBIK_OK : hip_fail(e);
}

// How tbik_gemm_swiglu runs a shape (pure): the K split of the [M, 2 I] GEMM, and whether the unsplit case can end in
// the 128 x 128 tile's activation epilogue or has to pass gate and up through a 16-bit staging buffer.
enum { SWIGLU_FUSED = 0, SWIGLU_SPLIT = 1, SWIGLU_STAGED = 2 };
static int swiglu_route(int dtype, int M, int I, int K, int sl, int ns, int *split) {
    const int N = 2 * I;
    GemmArgs probe{nullptr, K, nullptr, N, nullptr, nullptr, I, dtype, M, N, K, sl, ns, 1, dtype, 0};
    probe.P = *split = internal_split(M, N, K, ns);
    if (*split > 1) return pick_variant(probe, tile_rows(M, N)) != VARIANT_REFERENCE ? SWIGLU_SPLIT : SWIGLU_STAGED;
    probe.swiglu = 1;
    return (tile_rows(M, N) == 128 && g_forced_variant.load() == VARIANT_AUTO && gemm_tiled_supports(probe, VARIANT_T128))
               ? SWIGLU_FUSED : SWIGLU_STAGED;
}

size_t tbik_gemm_swiglu_workspace_bytes(int M, int I, int K, int leaf, int k_first) {
    int sl, ns, split;
    if (I <= 0 || I > 0x3fffffff || check_tree(M, 2 * I, K, leaf, k_first, 1, &sl, &ns) != TBIK_OK) return 0;
    switch (swiglu_route(TBIK_BF16, M, I, K, sl, ns, &split)) {
        case SWIGLU_FUSED: return 0;
        case SWIGLU_SPLIT: return (size_t)split * (size_t)M * (size_t)(2 * I) * sizeof(float);
        default: return (((size_t)M * (size_t)(2 * I) * 2 + 255) & ~(size_t)255) + split_planes_bytes(M, 2 * I, internal_split(M, 2 * I, K, ns));
    }
}

int tbik_silu_mul(const void *gate, int64_t ldg, const void *up, int64_t ldu, void *act, int64_t lda,
                  tbik_dtype dtype, int M, int I, void *hip_stream) {
    if (M < 0 || I < 0) return TBIK_ERR_SHAPE;
    if (dtype != TBIK_BF16 && dtype != TBIK_F16) return TBIK_ERR_DTYPE;
    if (M == 0 || I == 0) return TBIK_OK;
    if (!gate || !up || !act) return TBIK_ERR_NULL;
    if (ldg < I || ldu < I || lda < I) return TBIK_ERR_SHAPE;
    hipError_t e = launch_silu_mul((const uint16_t *)gate, ldg, (const uint16_t *)up, ldu, (uint16_t *)act, lda, (int)dtype, M, I,
                                   (hipStream_t)hip_stream);
    return e == hipSuccess ? TBIK_OK : hip_fail(e);
}

int tbik_gemm_swiglu(const void *X, int64_t ldx, const void *W_gu, int64_t ldw, void *act, int64_t lda,
                     tbik_dtype dtype, int M, int I, int K, int leaf, int k_first,
                     void *workspace, size_t workspace_bytes, void *hip_stream) {
    if (I < 0 || I > 0x3fffffff || I % 8 != 0) return TBIK_ERR_SHAPE;
    const int N = 2 * I;
    int sl, ns;
    int rc = check_tree(M, N, K, leaf, k_first, 1, &sl, &ns);
    if (rc != TBIK_OK) return rc;
    if (dtype != TBIK_BF16 && dtype != TBIK_F16) return TBIK_ERR_DTYPE;
    if (M == 0 || I == 0) return TBIK_OK;
    rc = check_operands((int)dtype, X, ldx, W_gu, ldw, N, K);
    if (rc != TBIK_OK) return rc;
    if (ldx >= (1 << 22) || ldw >= (1 << 22)) return TBIK_ERR_SHAPE;
    if (!act) return TBIK_ERR_NULL;
    if (lda < I) return TBIK_ERR_SHAPE;
    if (!aligned(act, 2)) return TBIK_ERR_ALIGN;
    const size_t need = tbik_gemm_swiglu_workspace_bytes(M, I, K, leaf, k_first);
    if (need > 0 && (!workspace || workspace_bytes < need)) return TBIK_ERR_WORKSPACE;
    if (workspace && !aligned(workspace, 256)) return TBIK_ERR_ALIGN;

    hipStream_t s = (hipStream_t)hip_stream;
    int split;
    const int route = swiglu_route((int)dtype, M, I, K, sl, ns, &split);
    GemmArgs a{(const uint16_t *)X, ldx, (const uint16_t *)W_gu, ldw, nullptr, act, lda, (int)dtype, M, N, K, sl, ns, 1, (int)dtype, 0};
    hipError_t e;
    if (route == SWIGLU_FUSED) {
        a.swiglu = 1;
        e = launch_gemm_tiled(a, VARIANT_T128, s);
    } else if (route == SWIGLU_SPLIT) {
        a.partials = reinterpret_cast<float *>(workspace);
        a.Y = nullptr;
        a.P = split;
        e = launch_tiled(a, pick_variant(a, tile_rows(M, N)), s);
        if (e == hipSuccess) e = launch_tree_combine_swiglu(a.partials, split, (uint16_t *)act, lda, (int)dtype, M, I, s);
    } else {
        uint16_t *staged = reinterpret_cast<uint16_t *>(workspace);
        const size_t staged_bytes = ((size_t)M * (size_t)N * 2 + 255) & ~(size_t)255;
        rc = gemm((int)dtype, X, ldx, W_gu, ldw, staged, N, (int)dtype, M, N, K, leaf, k_first,
                  reinterpret_cast<char *>(workspace) + staged_bytes, workspace_bytes - staged_bytes, hip_stream);
        if (rc != TBIK_OK) return rc;
        e = launch_silu_mul(staged, N, staged + I, N, (uint16_t *)act, lda, (int)dtype, M, I, s);
    }
    return e == hipSuccess ? TBIK_OK : hip_fail(e);
}

int tbik_tree_allreduce(float *bufs, int P, int64_t n, void *hip_stream) {
    if (n < 0) return TBIK_ERR_SHAPE;
    if (P < 1 || !is_pow2(P) || P > TBIK_MAX_SHARDS) return TBIK_ERR_SHARDS;
    if (n == 0) return TBIK_OK;
    if (!bufs) return TBIK_ERR_NULL;
    if (!aligned(bufs, 16)) return TBIK_ERR_ALIGN;
    hipError_t e = launch_tree_allreduce(bufs, P, n, (hipStream_t)hip_stream);
    return e == hipSuccess ? TBIK_OK : hip_fail(e);
}

static int rmsnorm(int dtype, const void *x, const void *weight, void *y, int M, int H, float eps, void *hip_stream) {
    if (M < 0 || H <= 0 || H % 8 != 0 || H > 65536) return TBIK_ERR_SHAPE;
    if (M == 0) return TBIK_OK;
    if (!x || !weight || !y) return TBIK_ERR_NULL;
    if (!aligned(x, 16) || !aligned(weight, 16) || !aligned(y, 16)) return TBIK_ERR_ALIGN;
    hipError_t e = launch_rmsnorm((const uint16_t *)x, (const uint16_t *)weight, (uint16_t *)y, M, H, eps, dtype,
                                  (hipStream_t)hip_stream);
    return e == hipSuccess ? TBIK_OK : hip_fail(e);
}

int tbik_rmsnorm(const void *x, const void *weight, void *y, int M, int H, float eps, void *hip_stream) {
    return rmsnorm(TBIK_BF16, x, weight, y, M, H, eps, hip_stream);
}

int tbik_rmsnorm_f16(const void *x, const void *weight, void *y, int M, int H, float eps, void *hip_stream) {
    return rmsnorm(TBIK_F16, x, weight, y, M, H, eps, hip_stream);
}

static int attention(int dtype, const void *Q, const void *K, const void *V, void *O,
                     const int32_t *cu_seqlens_q, const int32_t *cu_seqlens_k, int batch, int max_seqlen_q, int max_seqlen_k,
                     int total_q, int total_k, int heads_q, int heads_kv, int head_dim,
                     int64_t q_stride, int64_t k_stride, int64_t v_stride, int64_t o_stride,
                     float scale, int causal, void *workspace, size_t workspace_bytes, void *hip_stream) {
    if (batch < 0 || max_seqlen_q < 0 || max_seqlen_k < 0 || total_q < 0 || total_k < 0 || heads_q <= 0 || heads_kv <= 0 ||
        head_dim <= 0)
        return TBIK_ERR_SHAPE;
    if (heads_q % heads_kv != 0 || heads_q > 65535 || batch > 65535) return TBIK_ERR_SHAPE;
    if (head_dim != 128) return TBIK_ERR_UNSUPPORTED;
    if (q_stride >= (1 << 24) || k_stride >= (1 << 24) || v_stride >= (1 << 24) || o_stride >= (1 << 24)) return TBIK_ERR_SHAPE;
    if (q_stride < (int64_t)heads_q * head_dim || o_stride < (int64_t)heads_q * head_dim ||
        k_stride < (int64_t)heads_kv * head_dim || v_stride < (int64_t)heads_kv * head_dim)
        return TBIK_ERR_SHAPE;
    if (batch == 0 || max_seqlen_q == 0 || total_q == 0) return TBIK_OK;
    if (!Q || !O || !cu_seqlens_q || !cu_seqlens_k) return TBIK_ERR_NULL;
    if (total_k > 0 && (!K || !V)) return TBIK_ERR_NULL;
    if (!aligned(Q, 16) || !aligned(K, 16) || !aligned(V, 16) || !aligned(O, 16) || !aligned(cu_seqlens_q, 4) ||
        !aligned(cu_seqlens_k, 4) || q_stride % 8 || k_stride % 8 || v_stride % 8 || o_stride % 8)
        return TBIK_ERR_ALIGN;
    if (max_seqlen_k > total_k) max_seqlen_k = total_k;          // no sequence has more keys than the call
    const size_t need = attention_workspace_required(batch, max_seqlen_q, max_seqlen_k, heads_q, heads_kv);     // more room may allow splits side by side
    if (need > 0 && (!workspace || workspace_bytes < need)) return TBIK_ERR_WORKSPACE;
    if (need > 0 && !aligned(workspace, 256)) return TBIK_ERR_ALIGN;
    AttnArgs a{(const uint16_t *)Q, (const uint16_t *)K, (const uint16_t *)V, (uint16_t *)O, dtype, cu_seqlens_q, cu_seqlens_k,
               batch, max_seqlen_q, max_seqlen_k, total_q, total_k, heads_q, heads_kv, q_stride, k_stride, v_stride, o_stride,
               scale, causal != 0, need > 0 ? workspace : nullptr, need > 0 ? workspace_bytes : 0};
    hipError_t e = launch_attention(a, (hipStream_t)hip_stream);
    return e == hipSuccess ? TBIK_OK : hip_fail(e);
}

int tbik_attention(const void *Q, const void *K, const void *V, void *O,
                   const int32_t *cu_seqlens_q, const int32_t *cu_seqlens_k, int batch, int max_seqlen_q, int max_seqlen_k,
                   int total_q, int total_k, int heads_q, int heads_kv, int head_dim,
                   int64_t q_stride, int64_t k_stride, int64_t v_stride, int64_t o_stride,
                   float scale, int causal, void *workspace, size_t workspace_bytes, void *hip_stream) {
    return attention(TBIK_BF16, Q, K, V, O, cu_seqlens_q, cu_seqlens_k, batch, max_seqlen_q, max_seqlen_k, total_q, total_k, heads_q,
                     heads_kv, head_dim, q_stride, k_stride, v_stride, o_stride, scale, causal, workspace, workspace_bytes,
                     hip_stream);
}

int tbik_attention_f16(const void *Q, const void *K, const void *V, void *O,
                       const int32_t *cu_seqlens_q, const int32_t *cu_seqlens_k, int batch, int max_seqlen_q, int max_seqlen_k,
                       int total_q, int total_k, int heads_q, int heads_kv, int head_dim,
                       int64_t q_stride, int64_t k_stride, int64_t v_stride, int64_t o_stride,
                       float scale, int causal, void *workspace, size_t workspace_bytes, void *hip_stream) {
    return attention(TBIK_F16, Q, K, V, O, cu_seqlens_q, cu_seqlens_k, batch, max_seqlen_q, max_seqlen_k, total_q, total_k, heads_q,
                     heads_kv, head_dim, q_stride, k_stride, v_stride, o_stride, scale, causal, workspace, workspace_bytes,
                     hip_stream);
}

size_t tbik_attention_workspace_bytes(int batch, int max_seqlen_q, int max_seqlen_k, int heads_q, int heads_kv) {
    return attention_workspace(batch, max_seqlen_q, max_seqlen_k, heads_q, heads_kv);
}

int tbik_set_attention_variant(int variant) { return set_attention_variant(variant) < 0 ? TBIK_ERR_DTYPE : TBIK_OK; }

size_t tbik_row_reduce_workspace_bytes(int M, int64_t V, tbik_rowop op) {
    if (op != TBIK_SUM && op != TBIK_MAX && op != TBIK_LOGSOFTMAX) return 0;
    // sized for the finer of the two input types (fp32 rows have twice the leaves of 16-bit rows)
    return row_reduce_workspace(M, V, TBIK_F32, (int)op);
}

static int combine_residual_rmsnorm(int dtype, const float *partials, int P, const void *residual, const void *weight,
                                    float eps, void *hidden, void *normed, int M, int H, void *hip_stream) {
    if (M < 0 || H <= 0 || H % 8 != 0 || H > 65536) return TBIK_ERR_SHAPE;
    if (P < 1 || !is_pow2(P) || P > TBIK_MAX_SHARDS) return TBIK_ERR_SHARDS;
    if (P > 16) return TBIK_ERR_UNSUPPORTED;
    if (M == 0) return TBIK_OK;
    if (!partials || !residual || !weight || !hidden || !normed) return TBIK_ERR_NULL;
    if (!aligned(partials, 16) || !aligned(residual, 16) || !aligned(weight, 16) || !aligned(hidden, 16) || !aligned(normed, 16))
        return TBIK_ERR_ALIGN;
    if (normed == hidden || normed == residual) return TBIK_ERR_SHAPE;      // only hidden may share residual's buffer
    hipError_t e = launch_combine_residual_rmsnorm(partials, P, (const uint16_t *)residual, (const uint16_t *)weight,
                                                   (uint16_t *)hidden, (uint16_t *)normed, M, H, eps, dtype,
                                                   (hipStream_t)hip_stream);
    return e == hipSuccess ? TBIK_OK : hip_fail(e);
}

int tbik_combine_residual_rmsnorm(const float *partials, int P, const void *residual, const void *weight, float eps,
                                  void *hidden, void *normed, int M, int H, void *hip_stream) {
    return combine_residual_rmsnorm(TBIK_BF16, partials, P, residual, weight, eps, hidden, normed, M, H, hip_stream);
}

int tbik_combine_residual_rmsnorm_f16(const float *partials, int P, const void *residual, const void *weight, float eps,
                                      void *hidden, void *normed, int M, int H, void *hip_stream) {
    return combine_residual_rmsnorm(TBIK_F16, partials, P, residual, weight, eps, hidden, normed, M, H, hip_stream);
}

int tbik_row_reduce(const void *x, tbik_dtype x_dtype, void *out, tbik_rowop op, int M, int64_t V,
                    void *workspace, size_t workspace_bytes, void *hip_stream) {
    if (x_dtype != TBIK_F32 && x_dtype != TBIK_BF16 && x_dtype != TBIK_F16) return TBIK_ERR_DTYPE;
    if (op != TBIK_SUM && op != TBIK_MAX && op != TBIK_LOGSOFTMAX) return TBIK_ERR_DTYPE;
    const int epl = (x_dtype == TBIK_F32) ? 4 : 8;
    if (M < 0 || V <= 0 || V % epl != 0) return TBIK_ERR_SHAPE;
    if (M == 0) return TBIK_OK;
    if (!x || !out) return TBIK_ERR_NULL;
    if (!aligned(x, 16) || !aligned(out, op == TBIK_LOGSOFTMAX ? 16 : 4)) return TBIK_ERR_ALIGN;
    const size_t need = row_reduce_workspace(M, V, (int)x_dtype, (int)op);
    if (!workspace || workspace_bytes < need) return TBIK_ERR_WORKSPACE;
    if (!aligned(workspace, 256)) return TBIK_ERR_ALIGN;
    hipError_t e = launch_row_reduce(x, (int)x_dtype, out, (int)op, M, V, workspace, (hipStream_t)hip_stream);
    return e == hipSuccess ? TBIK_OK : hip_fail(e);
}

int tbik_row_reduce_static(const void *x, tbik_dtype x_dtype, void *out, tbik_rowop op, int M, int64_t V, void *hip_stream) {
    if (x_dtype != TBIK_F32 && x_dtype != TBIK_BF16 && x_dtype != TBIK_F16) return TBIK_ERR_DTYPE;
    if (op != TBIK_SUM && op != TBIK_MAX && op != TBIK_LOGSOFTMAX) return TBIK_ERR_DTYPE;
    const int epl = (x_dtype == TBIK_F32) ? 4 : 8;
    if (M < 0 || V <= 0 || V % epl != 0) return TBIK_ERR_SHAPE;
    if (M > 0) {
        if (!x || !out) return TBIK_ERR_NULL;
        if (!aligned(x, 16) || !aligned(out, op == TBIK_LOGSOFTMAX ? 16 : 4)) return TBIK_ERR_ALIGN;
        if (row_reduce_workspace(M, V, (int)x_dtype, (int)op) > (size_t)TBIK_STATIC_SCRATCH_BYTES) return TBIK_ERR_WORKSPACE;
    }
    hipError_t e = launch_row_reduce_static(x, (int)x_dtype, out, (int)op, M, V, (hipStream_t)hip_stream);
    return e == hipSuccess ? TBIK_OK : hip_fail(e);
}

int tbik_set_row_wait_limit(int polls) { return set_row_wait_limit(polls); }

int tbik_set_gemm_variant(int variant) {
    if (variant < 0 || variant >= VARIANT_COUNT) return TBIK_ERR_UNSUPPORTED;
    g_forced_variant.store(variant);
    return TBIK_OK;
}

int tbik_gemm_route(tbik_dtype x_dtype, int scaled, int M, int N, int K, int leaf, int k_first, int route[8]) {
    int sl, ns;
    int rc = check_tree(M, N, K, leaf, k_first, 1, &sl, &ns);
    if (rc != TBIK_OK) return rc;
    const int t = (int)x_dtype;
    const bool wide = t == TBIK_F32 || t == TBIK_BF16 || t == TBIK_F16;
    if (!route) return TBIK_ERR_NULL;
    if (!wide && !is_fp8(t) && t != TBIK_MXFP4 && t != TBIK_FP6_E2M3 && t != TBIK_FP6_E3M2) return TBIK_ERR_DTYPE;
    if (!wide && sl % 64 != 0) return TBIK_ERR_SHAPE;
    std::fill(route, route + 8, 0);
    if (M == 0 || N == 0) return TBIK_OK;
    const bool mx = !wide && (scaled || !is_fp8(t));
    const int64_t ld = wide ? K : t == TBIK_MXFP4 ? K / 2 : is_fp8(t) ? K : (int64_t)K * 3 / 4;     // dense rows of X
    uint8_t *const dense = reinterpret_cast<uint8_t *>((uintptr_t)256);                             // asked for its alignment only
    const Mxfp4Scales sc{dense, (K / 32 + 3) / 4 * 4, dense, (K / 32 + 3) / 4 * 4};
    int *out = route;
    auto note = [&](int, int m, TilePlan plan) {
        GemmArgs a{reinterpret_cast<const uint16_t *>(dense), ld, reinterpret_cast<const uint16_t *>(dense), wide ? N : ld, nullptr, dense, N,
                   t, m, N, K, sl, ns, 1, t, 0};
        out[0] = m;
        if (wide) {
            GemmArgs probe = a;
            probe.P = plan.split;
            const int v = pick_variant(probe, plan.rows);
            out[1] = v == VARIANT_REFERENCE ? KERNEL_REFERENCE : KERNEL_TILED;
            out[2] = v == VARIANT_T128 ? 128 : v == VARIANT_T96 ? 96 : v == VARIANT_T64 && t != TBIK_F32 ? 64 : 32;
        } else {
            out[1] = low_bit_kernel(a, mx ? &sc : nullptr, plan.split);
            out[2] = plan.rows;
        }
        out[3] = plan.split;
        if (out[1] != KERNEL_TILED) out[2] = out[3] = 0;
        out += 4;
        return hipSuccess;
    };
    if (t == TBIK_F32) (void)note(0, M, {0, f32_plan(M, N, K, ns).split});
    else (void)in_pieces(wide ? OPERANDS_16BIT : t == TBIK_MXFP4 ? OPERANDS_MXFP4 : !is_fp8(t) ? OPERANDS_MXFP6 : mx ? OPERANDS_MXFP8 : OPERANDS_FP8,
                         M, N, K, ns, SIZE_MAX, note);
    return TBIK_OK;
}

const char *tbik_variant_name(int variant) {
    return (variant >= 0 && variant < VARIANT_COUNT) ? kVariantNames[variant] : nullptr;
}

const char *tbik_status_string(int status) {
    switch (status) {
        case TBIK_OK: return "ok";
        case TBIK_ERR_NULL: return "null pointer";
        case TBIK_ERR_SHAPE: return "illegal shape or tree parameters";
        case TBIK_ERR_SHARDS: return "illegal shard count";
        case TBIK_ERR_DTYPE: return "illegal dtype or op";
        case TBIK_ERR_ALIGN: return "misaligned pointer or leading dimension";
        case TBIK_ERR_WORKSPACE: return "workspace missing or too small";
        case TBIK_ERR_UNSUPPORTED: return "unsupported";
        case TBIK_ERR_HIP: return "HIP runtime error";
        default: return "unknown status";
    }
}

int tbik_last_hip_error(void) { return g_last_hip_error.load(); }

const char *tbik_version(void) { return "tbik-gfx950 0.1"; }

}  // extern "C"
