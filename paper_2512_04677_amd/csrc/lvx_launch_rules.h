// Which kernel a call takes: the tile of a matrix product, of a convolution step, the workgroup form of the attention.  Rules on sizes
// only, in plain host C++ with no GPU types, so that they can be evaluated for any size without a GPU.
#pragma once
#include <stddef.h>
#include <stdint.h>

typedef uint16_t bf16_t;  // raw bf16 bits in memory

constexpr int LVX_NUM_CU = 256;

// Rounds of the chip that so many workgroups take, one per compute unit.
static inline long lvx_rounds(long workgroups) { return (workgroups + LVX_NUM_CU - 1) / LVX_NUM_CU; }

// ---- matrix products -----------------------------------------------------------------------------------------------------------
// Several projections of the same activations in one GEMM launch: segment i owns the column tiles from tn_begin on (filled in
// by the launcher) and has its own weight matrix [N][ldw], output (bf16, or fp32 if f32), output row stride and width.
#define LVX_GEMM_MAX_SEGS 16
struct lvx_gemm_seg_t {
    const bf16_t *W;
    void *C;
    int64_t ldc;
    int32_t N, tn_begin, f32, ld_sumsq;
    // NULL, or [M][ld_sumsq] floats: besides the bf16 store, the kernel leaves for each row the sums of squares (taken on the fp32
    // accumulators) of lvx_gemm_sumsq_parts(M, N, K) equal groups of columns: the partial sums of a row's RMS, added up in a fixed
    // order by the consumer (no atomics: results stay bit-reproducible).  One segment only, N % 64 == 0.
    float *sumsq;
};
#define LVX_GEMM_MAX_SUMSQ_PARTS(N_) ((N_) / 16)
// Who decides how many K groups a launch sums in (its order of summation): the first product as if it were launched alone, unless that
// would cost its company too much (see lvx_gemm_pick_tile), the launch as a whole (products that are only ever launched together), or
// nobody: one group (products launched with more or fewer others, like the context's projections of a group of layers).
enum { LVX_GEMM_ORDER_FIRST = 0, LVX_GEMM_ORDER_LAUNCH = 1, LVX_GEMM_ORDER_ONE = 2 };
struct lvx_gemm_segs_t {
    int32_t n, order;
    lvx_gemm_seg_t s[LVX_GEMM_MAX_SEGS];
};

// The small tiles, widest first: id, BM, BN, WM, WN, NST, KG, columns per partial sum of squares (a wave's columns; 16 where K
// groups reduce in LDS), and the time in microseconds that a compute unit needs per slab of such a tile (measured while the
// tiles stream their weights from HBM; a slab is 128 bytes of every row in bf16 and in FP8 alike).
#define LVX_GEMM_SMALL_TILES(X_)          \
    X_(0, 64, 128, 2, 4, 6, 1, 32, 0.42f) \
    X_(1, 64, 64, 2, 4, 4, 1, 16, 0.31f)  \
    X_(2, 32, 64, 1, 4, 5, 2, 16, 0.235f) \
    X_(3, 32, 32, 1, 2, 4, 4, 16, 0.16f)
// 128 x 256 and 128 x 192 tiles, per slab and compute unit, measured on kernels of such tiles.  lvx_gemm_wide_kernel has replaced those; it works such tiles
// as halves of its own in the same time or less (LVX_GEMM_WIDE_US).  The rules down to lvx_gemm_plan still compare the small tiles with them, which
// says where a product is small and in how many K groups it is summed; lvx_gemm_choose then puts what falls to them on the wide kernel.
#define LVX_GEMM_SLAB_US_128X256 0.80f
#define LVX_GEMM_SLAB_US_128X192 0.66f
enum { LVX_GEMM_TILE_128X256 = -1, LVX_GEMM_TILE_128X192 = -2 };

// Column tiles of width bn of the product(s).
static inline long lvx_gemm_col_tiles(const lvx_gemm_segs_t *segs, int N, int bn) {
    if (segs == nullptr || segs->n == 0) return (N + bn - 1) / bn;
    long t = 0;
    for (int i = 0; i < segs->n; ++i) t += (segs->s[i].N + bn - 1) / bn;
    return t;
}

// Which small tile to use, or one of the large ones (128 x 192 only if `narrow` says that the caller can use it, and only where that takes at
// most LVX_GEMM_NARROW_MAX of the 128 x 256 tiles' time: 174 shapes at 0.825 by the rule, the same number of rounds, ran in 0.87 of it,
// but nine at 0.99, six rounds for five, in 1.015): the one whose rounds of the
// chip (a compute unit that gets two tiles needs twice the time, whether one after the other or side by side) times slabs
// times time per slab is least.  A small tile costs more per flop but less per tile, so it wins exactly where the larger ones do
// not fill the chip: at N = K = 2560 32 x 32 up to 96 rows, 32 x 64 up to 192, 64 x 64 up to 384, 64 x 128 up to 768, 128 x 192 up to 2304.
// The number of K groups fixes the order in which a product is summed; segs->order says who decides it (see lvx_gemm_segs_t).
// LVX_GEMM_ORDER_FIRST takes the groups that suit the first product alone, so that its bits are those of a launch of its own, as long as
// the launch then costs at most LVX_GEMM_FIRST_MAX of the 128 x 256 launch of both, and one group otherwise: a narrow product's K groups
// have only the smallest tiles, and a wide second product in those took up to six times as long (1170 x (256 + 5120) x 5120: 68 us in 128 x
// 256 tiles, 182 in 32 x 64; 4680 x (16 + 13824) x 5120: 541 and 2129).  The line lies below 1 because each further round of small tiles
// also pays a start and a reduction that the time per slab does not hold: 48 x (416 + 9712) x 384, 0.80 by the rule, 9.3 and 10.5.
#define LVX_GEMM_FIRST_MAX 0.75
#define LVX_GEMM_NARROW_MAX 0.97
static inline int lvx_gemm_pick_tile(const lvx_gemm_segs_t *segs, int M, int N, int n_slabs, bool narrow = false, double *cost_us = nullptr) {
    const bool many = segs != nullptr && segs->n > 0;
    const int order = many ? segs->order : LVX_GEMM_ORDER_LAUNCH;
    int groups = order == LVX_GEMM_ORDER_ONE ? 1 : 0, best = LVX_GEMM_TILE_128X256;  // 0: not decided yet
    // pass 0: the first product alone decides the groups; 1: the tile; 2: the tile once more, for one group
    for (int pass = order == LVX_GEMM_ORDER_FIRST ? 0 : 1, last = 1; pass <= last; ++pass) {
        const lvx_gemm_segs_t *sg = pass == 0 ? nullptr : segs;
        const int n = many ? segs->s[0].N : N;
        auto rounds = [&](int bm, int bn) { return (double)lvx_rounds((long)((M + bm - 1) / bm) * lvx_gemm_col_tiles(sg, n, bn)); };
        const double large_cost = rounds(128, 256) * n_slabs * LVX_GEMM_SLAB_US_128X256;
        double best_cost = groups <= 1 ? large_cost : 1e30;
        int best_groups = 1;
        best = LVX_GEMM_TILE_128X256;
        if (narrow && groups <= 1 && rounds(128, 192) * n_slabs * LVX_GEMM_SLAB_US_128X192 < LVX_GEMM_NARROW_MAX * best_cost)
            best_cost = rounds(128, 192) * n_slabs * LVX_GEMM_SLAB_US_128X192, best = LVX_GEMM_TILE_128X192;
#define LVX_TILE_COST(ID_, BM_, BN_, WM_, WN_, NST_, KG_, PC_, US_)                                         \
    if (groups == 0 || KG_ == groups) {                                                                     \
        const double c_ = rounds(BM_, BN_) * ((n_slabs + KG_ - 1) / KG_ * KG_) * US_;                       \
        if (c_ < best_cost) best_cost = c_, best = ID_, best_groups = KG_;                                  \
    }
        LVX_GEMM_SMALL_TILES(LVX_TILE_COST)
#undef LVX_TILE_COST
        groups = best_groups;
        if (pass == 1 && order == LVX_GEMM_ORDER_FIRST && groups > 1 && best_cost > LVX_GEMM_FIRST_MAX * large_cost) groups = 1, last = 2;
        if (cost_us != nullptr) *cost_us = best_cost;
    }
    return best;
}

// Rows of a product that fill whole rounds of the chip as 128 x 256 tiles, the rest (*rest_tile) going to a small tile in a second launch; 0: all
// rows in one launch.  A product of 260 such tiles on 256 compute units takes two rounds, the second nearly empty.  Chosen where the sum of both, and a
// launch's LVX_GEMM_LAUNCH_US, is less than best_us, the time of the single launch.  Only tiles without K groups: these sum in the order of the
// wide kernel and with its matrix instructions, in bf16 and in FP8, so a row's bits are the same on either side of the split.  Partial sums of squares need one
// column grouping for all rows, so such a product is not split.  Nor is one of more than LVX_GEMM_SPLIT_ROUNDS whole rounds: compute units drift apart from round to
// round, so that the last, partial one begins before the one before it has ended (one whole round 0.77 to 0.89 of the single launch's time on a kernel of 128 x 256
// tiles, four 0.91 to 1.01, five 0.93 to 1.00, six to ten 0.98 to 1.10).  The wide kernel's halves make a last round cheaper, so most of these products now
// run whole on it (1560 x 5120 x 13824 306 us in 128 x 256 tiles, 234 split, 190 now); see lvx_gemm_choose.
#define LVX_GEMM_LAUNCH_US 3.0
#define LVX_GEMM_SPLIT_ROUNDS 5
static inline int lvx_gemm_split_rows(const lvx_gemm_segs_t *segs, int M, int N, int n_slabs, double best_us, int *rest_tile) {
    const bool many = segs != nullptr && segs->n > 0;
    if (many && segs->s[0].sumsq != nullptr) return 0;
    const int n = many ? segs->s[0].N : N;
    const long cols = lvx_gemm_col_tiles(segs, n, 256), total = (long)((M + 127) / 128) * cols, rounds = total / LVX_NUM_CU;
    const int m1 = (int)(rounds * LVX_NUM_CU / cols * 128);
    if (m1 == 0 || m1 >= M || rounds > LVX_GEMM_SPLIT_ROUNDS) return 0;
    auto cost = [&](int m, int bm, int bn, double us) { return (double)lvx_rounds((long)((m + bm - 1) / bm) * lvx_gemm_col_tiles(segs, n, bn)) * n_slabs * us; };
    double best = best_us - cost(m1, 128, 256, LVX_GEMM_SLAB_US_128X256) - LVX_GEMM_LAUNCH_US;
    int tile = LVX_GEMM_TILE_128X256;
#define LVX_TILE_COST(ID_, BM_, BN_, WM_, WN_, NST_, KG_, PC_, US_) \
    if (KG_ == 1 && cost(M - m1, BM_, BN_, US_) < best) best = cost(M - m1, BM_, BN_, US_), tile = ID_;
    LVX_GEMM_SMALL_TILES(LVX_TILE_COST)
#undef LVX_TILE_COST
    *rest_tile = tile;
    return tile < 0 ? 0 : m1;
}
static inline int lvx_gemm_part_cols(int tile) {
#define LVX_TILE_PART(ID_, BM_, BN_, WM_, WN_, NST_, KG_, PC_, US_) \
    if (tile == ID_) return PC_;
    LVX_GEMM_SMALL_TILES(LVX_TILE_PART)
#undef LVX_TILE_PART
    return 64;
}

// What the rules above make of a product: the tile, and the rows m1 in whole rounds of 128 x 256 tiles before it (0: the tile takes all rows).
struct lvx_gemm_plan_t {
    int tile, m1;
    double us;  // the single launch's time by the rule above
};
static inline lvx_gemm_plan_t lvx_gemm_plan(const lvx_gemm_segs_t *segs, int M, int N, int n_slabs, bool narrow) {
    lvx_gemm_plan_t p = {0, 0, 0};
    p.tile = lvx_gemm_pick_tile(segs, M, N, n_slabs, narrow, &p.us);
    int rest = p.tile;
    if (p.tile < 0) p.m1 = lvx_gemm_split_rows(segs, M, N, n_slabs, p.us, &rest);
    if (p.m1 > 0) p.tile = rest;
    return p;
}

// ---- 256 x 256 tiles (lvx_gemm_wide.h) -------------------------------------------------------------------------------------------
// The wide kernel's tiles have 256 rows, or as halves 128: M rows are lvx_wide_full_rows row tiles of 256 and, if at most 128 rows remain, one of 128;
// the first n_large of the 256-row tiles are taken whole, the others as two halves.
static inline int lvx_wide_full_rows(int M) { return M / 256 + (M % 256 > 128 ? 1 : 0); }
static inline long lvx_wide_halves(int M, long cols, long n_large) {
    const long full = lvx_wide_full_rows(M);
    return 2 * (full * cols - n_large) + ((M + 255) / 256 - full) * cols;
}

// Time by the rule of a launch with n_large whole tiles, slab by slab.  A whole tile takes 1.35 us a slab while all compute units have one (the
// chip is held by its power: 256 x 256 x 64 on 256 units in that time are 1.59 PFLOP/s) and down to 1.04 while half of them idle; a half
// 0.80, and up to 0.99 on the few units left beside a round of whole tiles that draws the power of the chip alone.  Whole tiles start
// first, each unit takes the next tile when it is free.  600 products, bf16 and FP8, 600 to 8000 rows, each with none, all and whole rounds of
// whole tiles: the choice by the rule takes 0.1 % longer on average than the fastest of them.  2048 x 8192 x 5120 as 256 whole tiles 116 us, as
// 512 halves 147; 4680 x 5120 x 5120 as 256 + 228 halves 174, 360 + 20 199, 740 halves 198; 1560 x 13824 x 5120 as 256 + 190 183, 324 + 54 204;
// 2150 x 7656 x 4224 as 510 halves 114, 240 + 30 135.
// (lvx_wide_us_t: a whole tile on a busy chip and beside idle units, a half.)
struct lvx_wide_us_t {
    double whole, alone, half;
};
// Tiles of 256 x 64 fn, fn = 2, 3, 4.
constexpr lvx_wide_us_t LVX_GEMM_WIDE_US[3] = {{0.82, 0.68, 0.52}, {1.05, 0.80, 0.64}, {1.35, 1.04, LVX_GEMM_SLAB_US_128X256}};
static inline double lvx_wide_slab_us(int M, long cols, long n_large, const lvx_wide_us_t &us = LVX_GEMM_WIDE_US[2]) {
    const long busy = n_large % LVX_NUM_CU, halves = lvx_wide_halves(M, cols, n_large);
    const double whole = (double)(n_large / LVX_NUM_CU) * us.whole;
    if (busy == 0) return whole + lvx_rounds(halves) * us.half;
    const double most = LVX_NUM_CU / 2, last = us.alone + (busy > most ? (us.whole - us.alone) * (busy - most) / most : 0.0);
    // the last whole tiles take `busy` units for `last`, the other units begin the halves meanwhile: the first end of a half on either kind of
    // unit by which all of them are done
    const double beside = us.half + (busy > 208 ? 0.005 * us.half * (busy - 208) : 0.0);
    const long idle = LVX_NUM_CU - busy;
    long early = 0, late = 0;
    double end = last;
    while (idle * early + busy * late < halves) {
        const double a = (early + 1) * beside, b = last + (late + 1) * us.half;
        if (a <= b) ++early;
        else ++late;
        const double t = a <= b ? a : b;
        if (t > end) end = t;
    }
    return whole + end;
}
// How many whole tiles are best: all, whole rounds of the chip, one round less, or none.
static inline long lvx_wide_pick(int M, long cols, double *slab_us, const lvx_wide_us_t &us = LVX_GEMM_WIDE_US[2]) {
    const long total = lvx_wide_full_rows(M) * cols, rounds = total / LVX_NUM_CU * LVX_NUM_CU;
    long best = 0;
    double best_us = lvx_wide_slab_us(M, cols, 0, us);
    const long offer[3] = {rounds - LVX_NUM_CU, rounds, total};
    for (int i = 0; i < 3; ++i)
        if (offer[i] > 0 && lvx_wide_slab_us(M, cols, offer[i], us) <= best_us) best = offer[i], best_us = lvx_wide_slab_us(M, cols, offer[i], us);
    *slab_us = best_us;
    return best;
}

// The launch of a product: lvx_gemm_plan, with the wide tiles (256 x 64 fn and their halves) where they are in reach.  wide_rows: the rows that the
// wide kernel takes, n_large whole tiles among them; the rows behind go to `tile` (m1 = wide_rows) or there are none.  Where the plan is
// one of the large tiles (128 x 256 or 128 x 192), the wide kernel takes all rows.  Rows split off give way where it takes no longer by the rule.  Small
// tiles for all rows stay: those with K groups fix the order of summation, and of those without only two rounds of 64 x 64 tiles beside one of 256 x 128
// halves would give way, but two such tiles share a compute unit (29 products in bf16 0.79 to 1.01 of the halves' time, mean 0.92, 24 in FP8 0.85 to 1.02,
// mean 0.95: 2110 x 936 x 3904 26.3 beside 29.2 us, 4335 x 432 x 1280 10.9 beside 12.9).  Narrower tiles, which move more bytes and power per product, are taken where they save a tenth by the
// rule, which means where they leave fewer compute units idle: below 0.90 110 products of 900 to 9000 rows took 0.70 to 1.06 of the time of
// 256-column tiles or of a 128 x 192 kernel of its own, mean 0.91 (1886 x 2560 x 2560 with residual 32.9 -> 31.4 us, 1560 x 5120 x 5120 with residual
// 86.7 -> 79.9, 1560 x 5120 x 13824 232 -> 190); from 0.90 to 1 they took 0.98 to 1.11, mean 1.03 (4680 x 15360 x 5120 505 -> 520).
// Partial sums of squares need columns by 64, so 256-column tiles, and a plan that leaves narrower ones stays.
#define LVX_WIDE_NARROWER 0.90
struct lvx_gemm_launch_t {
    int tile, wide_rows, fn, n_large;
};
static inline lvx_gemm_launch_t lvx_wide_best(const lvx_gemm_segs_t *segs, int M, int N, int fn_min, double *slab_us) {
    lvx_gemm_launch_t l = {LVX_GEMM_TILE_128X256, M, 4, 0};
    *slab_us = 1e30;
    for (int fn = 4; fn >= fn_min; --fn) {
        double us = 0.0;
        const long n_large = lvx_wide_pick(M, lvx_gemm_col_tiles(segs, N, 64 * fn), &us, LVX_GEMM_WIDE_US[fn - 2]);
        if (us < LVX_WIDE_NARROWER * *slab_us) *slab_us = us, l.fn = fn, l.n_large = (int)n_large;
    }
    return l;
}
static inline lvx_gemm_launch_t lvx_gemm_choose(const lvx_gemm_segs_t *segs, int M, int N, int n_slabs) {
    const bool many = segs != nullptr && segs->n > 0, sumsq = many && segs->s[0].sumsq != nullptr;
    const int n = many ? segs->s[0].N : N, fn_min = sumsq ? 4 : 2;
    const lvx_gemm_plan_t plan = lvx_gemm_plan(segs, M, N, n_slabs, !sumsq);
    double us = 0.0, part_us = 0.0;
    const lvx_gemm_launch_t wide = lvx_wide_best(segs, M, n, fn_min, &us);
    if (plan.m1 == 0) return plan.tile < 0 ? wide : lvx_gemm_launch_t{plan.tile, 0, 0, 0};
    lvx_gemm_launch_t split = lvx_wide_best(segs, plan.m1, n, fn_min, &part_us);
    split.tile = plan.tile;
    double rest_us = 0.0;
#define LVX_TILE_COST(ID_, BM_, BN_, WM_, WN_, NST_, KG_, PC_, US_) \
    if (plan.tile == ID_) rest_us = (double)lvx_rounds((long)((M - plan.m1 + BM_ - 1) / BM_) * lvx_gemm_col_tiles(segs, n, BN_)) * US_;
    LVX_GEMM_SMALL_TILES(LVX_TILE_COST)
#undef LVX_TILE_COST
    return us <= part_us + rest_us ? wide : split;
}

// ---- convolution ---------------------------------------------------------------------------------------------------------------
// The tiles with shared input rows: id, BM, BN, WM, WN, NST and the time in microseconds that a compute unit needs per stage (64
// channels of three taps)
#define LVX_CONV_ROW_TILES(X_)         \
    X_(0, 64, 64, 2, 4, 4, 0.70)       \
    X_(1, 128, 64, 4, 2, 3, 0.90)      \
    X_(2, 256, 64, 4, 2, 2, 1.48)      \
    X_(3, 192, 128, 4, 2, 2, 2.00)

// The kernel of a step of M output pixels (rows of W) and N channels, n_slabs 64-wide slabs of the contraction, is the
// one with the least rounds of the chip times slabs (or stages of three) times time of each: lvx_conv_large_kernel's 256 x 128 tiles
// where they fill the chip (C_out is 128 ... 512 in the decoder this serves; 128-wide column tiles waste nothing there), the tiles with shared
// input rows below that and where their rounds come out better, the 32 x 32 tile with four K groups for a few thousand outputs.  A pixel's
// bits must not depend on how many frames arrive with it: the first two kinds sum in one order, the K groups in another, so whether
// these are taken follows from max_m, the pixels of the longest step the layer takes.  Measured (us a step, before: 256 x 128 only or the
// linears' small tiles; 260 random layers and steps against 256 x 128 tiles everywhere: none slower, geometric mean 1.57): one 50 x 90 frame 384 -> 192 channels 119, 61 -> 42; four 25 x 45 frames 512 -> 512 146 -> 105; four 240 x 400
// 64 -> 64 199 -> 139; two 200 x 360 192 -> 96 238 -> 202.
enum { LVX_CONV_LARGE, LVX_CONV_ROWS, LVX_CONV_GROUPS };
struct lvx_conv_plan_t {
    int kind, tile;  // tile: of LVX_CONV_ROW_TILES or LVX_GEMM_SMALL_TILES
    double us;       // its time by the rule
};
static inline lvx_conv_plan_t lvx_conv_plan(int W, int N, int n_slabs, int M, int max_m) {
    lvx_conv_plan_t plan = {LVX_CONV_LARGE, 0, 0.0};
    for (int pass = 0; pass < 2; ++pass) {  // 0: K groups or not, at the longest step; 1: the tile, at this one
        const int m = pass == 0 ? max_m : M;
        const bool groups = pass == 1 && plan.kind == LVX_CONV_GROUPS;
        double best = 1e30;
        auto rounds = [&](long rows, int bm, int bn) { return (double)lvx_rounds((rows + bm - 1) / bm * ((N + bn - 1) / bn)); };
        auto offer = [&](int kind, int tile, double us) {
            if ((pass == 0 || (kind == LVX_CONV_GROUPS) == groups) && us < best) best = us, plan = {kind, tile, us};
        };
        offer(LVX_CONV_LARGE, 0, rounds(m, 256, 128) * n_slabs * 0.82);
        const long padded = (long)m / W * (W + 2);
#define LVX_TILE_COST(ID_, BM_, BN_, WM_, WN_, NST_, US_) offer(LVX_CONV_ROWS, ID_, rounds(padded, BM_, BN_) * (n_slabs / 3) * US_);
        LVX_CONV_ROW_TILES(LVX_TILE_COST)
#undef LVX_TILE_COST
#define LVX_TILE_COST(ID_, BM_, BN_, WM_, WN_, NST_, KG_, PC_, US_) \
    if (KG_ > 2) offer(LVX_CONV_GROUPS, ID_, rounds(m, BM_, BN_) * ((n_slabs + KG_ - 1) / KG_ * KG_) * US_);
        LVX_GEMM_SMALL_TILES(LVX_TILE_COST)
#undef LVX_TILE_COST
    }
    return plan;
}

// The kernel of a step: lvx_conv_plan, or tiles of 256 x 64 fn (fn 2, 3 or 4; lvx_gemm_wide.h) and their halves where these take at most
// LVX_CONV_WIDE_MAX of its time.  They sum in the order of the first two kinds, so a step may take them whatever the layer's other steps
// take; a layer of K groups keeps them.  Measured, us a step: four 100 x 180 frames 384 -> 384 channels 524 -> 463 (fn 3), four 127 x 85 64 -> 176 57
// -> 38, four 185 x 373 128 -> 304 655 -> 541, two 115 x 172 384 -> 200 218 -> 175 (fn 4), three 74 x 217 448 -> 288 377 -> 326.  34 of 91 random layers and steps
// lie below the line and took 0.66 to 0.97, mean 0.82; between it and 1.1 wide tiles took 0.88 to 1.08, mean 1.01.  Whole tiles of 256 x 192 beside a
// single round of 256 x 128: the rule prices both for a full chip, but 195 tiles on 256 units take 0.67 us a slab, not 0.82, and 130 wide ones their 0.76;
// 12 steps took 1.10 to 1.16 of the round's time (94 x 179 384 -> 384 137 us, 157 wide), so the round keeps them.
#define LVX_CONV_WIDE_MAX 0.94
struct lvx_conv_launch_t {
    lvx_conv_plan_t plan;
    int fn, n_large;  // fn 0: the plan
};
static inline lvx_conv_launch_t lvx_conv_choose(int W, int N, int n_slabs, int M, int max_m) {
    const lvx_wide_us_t us[3] = {{0.85, 0.70, 0.51}, {1.05, 0.76, 0.60}, {1.28, 0.94, 0.71}};  // fn 2, 3, 4
    lvx_conv_launch_t l = {lvx_conv_plan(W, N, n_slabs, M, max_m), 0, 0};
    const bool one_round = l.plan.kind == LVX_CONV_LARGE && lvx_rounds((long)((M + 255) / 256) * ((N + 127) / 128)) == 1;
    double best = LVX_CONV_WIDE_MAX * l.plan.us;
    for (int fn = 2; fn <= 4 && l.plan.kind != LVX_CONV_GROUPS; ++fn) {
        double slab = 0.0;
        const long n_large = lvx_wide_pick(M, (N + 64 * fn - 1) / (64 * fn), &slab, us[fn - 2]);
        if (one_round && fn == 3 && n_large > 0) continue;
        if (slab * n_slabs < best) best = slab * n_slabs, l.fn = fn, l.n_large = (int)n_large;
    }
    return l;
}

// ---- attention -----------------------------------------------------------------------------------------------------------------
#define LVX_KEY_TILE 64  // keys per V^T tile in the cache and per LDS stage of the attention kernel

// Whether a workgroup takes 128 queries and splits the keys over its halves instead of 256 queries.  A round of the chip with
// the split takes 0.62 to 0.66 of a round without (measured from 9 to 150 key tiles, head_dim 64 and 128: half the tiles per wave, but
// twice the K / V stream per tile), up to 7 key tiles 0.69 to 0.85 (the exchange at the end is the same for every length), so it pays
// where the smaller workgroups need less than half, or a third, as many more rounds: always
// while they fit one round, e.g. 12 heads x 1170 queries x 6240 keys 134 -> 90 us, but 20 x 1886 x 8487 (160 workgroups become 300)
// 191 -> 236 us, and 24 x 3441 x 187 (three rounds for two) 19.8 -> 21.3.  A last query tile that leaves every SIMD to a single wave, or most
// SIMDs idle, takes about half the time at head_dim 128 (not at 64, where fewer MFMAs stand against the same softmax), so where it alone begins a round it counts for half of one (32 x 2142 x 1851, 79 rows behind one
// whole round: 90 us, 96 split; 24 x 4118 x 3072, 22 rows behind three rounds of the split form: 155, 192 split; 22 x 2823 x 2136, 7 rows: 114,
// 77 split).  With few key tiles a workgroup's start and end weigh more than its rows: the split form's last tile counts in full (24 x 2712 x
// 192: 18.1 us, 20.5 split).  Up to 128 queries half of the waves idle without the split; with less than 8 key tiles the exchange then
// costs what it saves (9.3 against 10.2 us at 4 tiles, 15.1 against 14.4 at 9).
static inline bool lvx_attention_splits_keys(int n_q, int H, int n_keys, int head_dim) {
    const bool few_tiles = n_keys <= 7 * LVX_KEY_TILE;
    if (n_q <= 128 && few_tiles) return false;
    auto rounds = [&](int qt) {
        const long full = n_q / qt, last = n_q % qt, whole = lvx_rounds(full * H), all = lvx_rounds((full + (last > 0)) * H);
        if (full == 0 || last > (qt == 256 ? 128 : 32)) return (double)all;
        if (few_tiles) return (double)(qt == 256 && last <= 64 ? whole : all);
        return head_dim == 64 ? (double)all : 0.5 * (whole + all);
    };
    return (few_tiles ? 0.74 : 0.65) * rounds(128) < rounds(256);
}

// Whether workgroups of 16 queries whose waves each take key tiles of their own (lvx_attention_few_kernel) serve the call: where all of them are on
// the chip at once (as many to a compute unit as its LDS holds, at most 4) and a wave has at most six tiles of head_dim 128 (twelve of 64).  Up to
// 256 of them take 6.6 us and 0.35 (0.22 at head_dim 64) a tile: 105 x 4 heads x 560 keys 14.1 -> 8.8 us, 390 x 4 x 1300 20.3 (over workgroups)
// -> 16.2, x 72 10.3 -> 6.6, 105 x 4 x 40 with the query norm 8.7 -> 6.8; at 60 tiles 27.5 beside 27.9, at 85 36.9 beside 32.8.  Where a second round is needed each costs 4 us more: 320 x 22 tiles
// 26.6 beside 22.0, 513 x 3 tiles 19.5 beside 16.2.  Up to 128 queries of head_dim 64 with a single tile stay (6.5 beside 6.7; above 128 8.2 -> 6.6).
#define LVX_ATTN_FEW_WAVES 8
// A wave's K and V^T tile stand beside each other in LDS (then both are loaded at once), or one after the other in the same place: up to 128 KB.
constexpr bool lvx_attention_few_apart(int n_waves, int head_dim) { return n_waves * head_dim <= 512; }
static inline int lvx_attention_few_waves(int n_keys) {
    const int tiles = (n_keys + LVX_KEY_TILE - 1) / LVX_KEY_TILE;
    return tiles < LVX_ATTN_FEW_WAVES ? tiles : LVX_ATTN_FEW_WAVES;
}
static inline size_t lvx_attention_few_lds(int n_waves, int head_dim) {
    return (size_t)n_waves * (lvx_attention_few_apart(n_waves, head_dim) ? 2 : 1) * LVX_KEY_TILE * head_dim * 2;
}
static inline bool lvx_attention_few(int n_q, int H, int n_keys, int head_dim) {
    const long workgroups = ((long)n_q + 15) / 16 * H, together = 160 * 1024 / ((long)lvx_attention_few_lds(lvx_attention_few_waves(n_keys), head_dim) + 1024);
    if (head_dim == 64 && n_keys <= LVX_KEY_TILE && n_q <= 128) return false;
    return workgroups <= LVX_NUM_CU * (together < 4 ? together : 4) && (int64_t)n_keys * head_dim <= 48 * LVX_KEY_TILE * 128;
}

// Into how many ranges of keys the self-attention of a block is split over workgroups (1: none), and whether a workgroup then takes 128 queries
// with its range split once more over its halves (`halves`) instead of 256.  Few heads and queries leave compute units idle that the
// ranges fill, but each range writes its outputs in fp32 and a second kernel reads them: about 7 us more, and the ranges' bytes at 4.1 TB/s
// both ways.  Microseconds per tile of 64 keys: 256 queries 1.30 to 1.50 the more units work (head_dim 64: 1.08), 128 queries 0.88 (0.63).
// Measured, alone -> split: 12 heads x 1170 queries x 6240 keys 89 -> 59 (2 ranges, 128 queries), 8 x 1800 x 4200 59 -> 45, 16 x 1200 x 5400 78 -> 64
// (3 ranges, 256 queries), 20 x 1886 x 8487 175 -> 163, 4 x 390 x 1300 26 -> 21, head_dim 64, 8 x 900 x 4800 52 -> 28; no gain: 4 x 105 x
// 560 16 -> 17, 30 x 1800 x 6000 144 -> 168.  More than four ranges were never best.  Beyond 384 workgroups of 128 queries (256 queries where
// that is more, and none above 256 heads) no key count makes ranges the faster form by this rule: they need as many rounds for each range then as the
// undivided call needs for its share.  So no more rows than that take ranges, and no scratch is reserved for more.
#define LVX_ATTN_MAX_PARTS 4
#define LVX_ATTN_PARTS_WORKGROUPS 384
struct lvx_attn_split_t {
    int parts;
    bool halves;
};
// The most rows, n_q of them at most, whose keys may be split.
static inline int lvx_attention_parts_rows(int n_q, int H) {
    const int rows = H > LVX_NUM_CU ? 0 : 128 * (LVX_ATTN_PARTS_WORKGROUPS / H > 2 ? LVX_ATTN_PARTS_WORKGROUPS / H : 2);
    return n_q < rows ? n_q : rows;
}
static inline int lvx_attention_most_parts(int n_q, int H) { return lvx_attention_parts_rows(n_q, H) == n_q ? LVX_ATTN_MAX_PARTS : 1; }
static inline lvx_attn_split_t lvx_attention_parts(int n_q, int H, int n_keys, int head_dim) {
    const int most = lvx_attention_most_parts(n_q, H), tiles = (n_keys + LVX_KEY_TILE - 1) / LVX_KEY_TILE;
    auto time = [&](int parts, bool halves) {
        const long wgs = (long)(halves ? (n_q + 127) / 128 : (n_q + 255) / 256) * H * parts, busy = wgs < LVX_NUM_CU ? wgs : LVX_NUM_CU;
        const double tile = halves ? (head_dim == 64 ? 0.63 : 0.88) : (head_dim == 64 ? 1.08 : 1.30 + 0.2 * busy / LVX_NUM_CU);
        const double ranges = parts > 1 ? 7.0 + parts * 8.0 * n_q * H * head_dim / 4.1e6 : 0.0;
        return (double)lvx_rounds(wgs) * ((tiles + parts - 1) / parts) * tile + 5.0 + ranges;
    };
    const double alone = time(1, lvx_attention_splits_keys(n_q, H, n_keys, head_dim));
    lvx_attn_split_t best = {1, false};
    double best_us = 0.94 * alone;
    for (int parts = 2; parts <= most && parts <= tiles; ++parts)
        for (int halves = 0; halves < 2; ++halves)
            if (time(parts, halves != 0) < best_us) best_us = time(parts, halves != 0), best = {parts, halves != 0};
    return best;
}
// Bytes of the ranges' outputs, references and sums, as many as there can be of them.
static inline size_t lvx_attention_scratch_bytes(int n_q, int H, int head_dim) {
    const size_t most = (size_t)lvx_attention_most_parts(n_q, H);
    return most <= 1 ? 0 : most * n_q * H * ((size_t)head_dim * 4 + 8);
}
