// Which tiles, slices and workspace a product takes: plain C++ on sizes alone, so that a test compiles it on the host and asks
// it.  mfma.hip and plain.hip launch what is planned here.
#pragma once
#include <math.h>
#include <stddef.h>
#include <stdint.h>

#include <initializer_list>

#include "../../include/rmm.h"

// (hidden: the plans that plan_pass remembers belong to one library)
namespace rmm __attribute__((visibility("hidden"))) {

inline int64_t tiles_of(int64_t m, int64_t n, int64_t bm, int64_t bn) { return ((m + bm - 1) / bm) * ((n + bn - 1) / bn); }

// Tile a plain product runs with (typedefs of mfma_kernels.hpp) and a sketch product's kernel.
enum { GEMM_LARGE = 0, GEMM_WIDE = 1, GEMM_SPLIT = 2, GEMM_MID = 3, GEMM_FLAT = 4, GEMM_SMALL = 5, GEMM_FEW = 6, GEMM_COMPACT = 7 };
enum { SK_NARROW = 0, SK_WIDE = 1, SK_WIDE64 = 2, SK_MID64 = 3, SK_MID = 4, SK_NARROW64 = 5 };
struct TileEdges {
    int64_t bm, bn;
};
constexpr TileEdges kGemmTiles[] = {{256, 256}, {128, 256}, {128, 128}, {128, 128}, {64, 128}, {64, 64}, {32, 32}, {128, 128}};
constexpr int64_t kFewSingle = 512;  // the longest contraction that is one step of every wave of few_tile
inline int64_t gemm_tiles(int cfg, int64_t m, int64_t n) { return tiles_of(m, n, kGemmTiles[cfg].bm, kGemmTiles[cfg].bn); }

// Work-groups of the column sums (colsum.hpp).
// 16-byte pieces per row and work-group: four where that still gives 96 work-groups, else one
// (measured at 16384 x 1024 bf16: 15 us with one, 21 with two, 41 with four).
inline int colsum_lpr(int64_t d, int64_t elem_bytes) { return d * elem_bytes / 16 >= 384 ? 4 : 1; }
inline int64_t colsum_blocks(int64_t d, int64_t elem_bytes) {
    const int64_t vecs = d * elem_bytes / 16, lpr = colsum_lpr(d, elem_bytes);
    return (vecs + lpr - 1) / lpr;
}
inline int64_t colsum_narrow_blocks(int64_t d) { return (d + 7) / 8; }

// Work-groups of the row norms of X and dY (row_norms.hpp): eight waves, one row of either per wave at a time; enough of them for the chip.
inline int row_norm_blocks(int64_t n) {
    const int64_t b = (n + 7) / 8;
    return (int)(b < 1024 ? b : 1024);
}

// The plain product of a paired launch: its tile (GEMM_LARGE, GEMM_WIDE, GEMM_MID or, with SK_NARROW64, GEMM_COMPACT; dX: see dx_cfg)
// and number of tiles.
struct PairPlain {
    int cfg, tiles;
};
// The sketch work-groups are put in front of the plain tiles when the sketch product is unsliced (few, long
// work-groups) or the plain product fills the chip at least once (256 tiles or more: measured 4 % faster at the
// RoBERTa-large shapes, 2-3 % slower where the plain product has 192 tiles and the sketch work-groups fill in behind).
inline bool sketch_goes_first(int64_t plain_tiles, int slices) { return slices == 1 || plain_tiles >= 256; }

inline bool mfma_shape_ok(int64_t n, int64_t d_in, int64_t d_out, int64_t k) {
    // 16-byte chunks need widths that are multiples of 8; a buffer descriptor spans up to 256 rows
    // of an operand with 32-bit byte offsets, so a row has to stay below 2^22 elements.  The token
    // count and the sketch size are not limited here (operands of 2 GiB and more are fine).
    (void)n, (void)k;
    const int64_t lim = (int64_t)1 << 22;
    return d_in % 8 == 0 && d_out % 8 == 0 && d_in < lim && d_out < lim;
}

// Time of a product on a menu of tiles, to choose between them (us, fitted to products from 256 x 384 to 16384 x 4096
// outputs and contractions from 51 to 4096): a launch, then rounds of 256 work-groups, each `fix` for the first loads and
// the writing of the tile and `step` for every 64 contraction elements.  Of the small tiles two share a compute unit: a
// full round of 512 takes 1.9 times the time of one of up to 256, one of 257 to 511 from 1.4 times on (`filled`, where other
// work-groups of the launch take the second places: 1.9 times too).
struct TileTime {
    double fix, step;
    bool shared;
};
inline double tile_us(const TileTime &t, int64_t tiles, int64_t kk, bool filled) {
    const int64_t rest = tiles % 512;
    const double rounds = !t.shared ? (double)((tiles + 255) / 256)
                                    : 1.9 * (double)(tiles / 512) + (rest == 0 ? 0.0 : rest <= 256 ? 1.0 : filled ? 1.9 : 1.4 + 0.5 * (double)(rest - 256) / 256.0);
    return 2.5 + rounds * (t.fix + (double)((kk + 63) / 64) * t.step);
}

// Tile of a plain product with an m x n output and contraction kk.  32 x 32 tiles whose contraction is shared by eight
// waves (few_tile) only while there are at most 512 of them.  256 x 256 tiles from 160 of them on whatever the model here
// says (a product alone in its launch is looked at again: gemm_cfg): they need half the bytes per flop of 128 x 128 tiles, which a full chip cannot bring into its LDS at MFMA rate.  And from 130 on
// where 128 x 128 tiles, with the `beside` other work-groups of the launch, go over two rounds (36 products from 516 to 660 of those:
// 0.73 to 1.02 of the time, 0.84 on average; with 455 to 510 of them 0.88 to 1.31).  (Times of the menu, and these 36 products, are from before
// the tiles' loops went through their LDS stages, which made 128 x 128 tiles faster, dX alone by 22 %, than 256 x 256 ones, 6 %.)
struct GemmChoice {
    int cfg;
    double us;
};
inline GemmChoice choose_gemm(int64_t m, int64_t n, int64_t kk, int64_t beside = 0) {
    const int64_t large = gemm_tiles(GEMM_LARGE, m, n);
    if (large >= 160 || (large >= 130 && gemm_tiles(GEMM_MID, m, n) + beside > 512))
        return GemmChoice{GEMM_LARGE, tile_us(TileTime{6.3, 1.405, false}, large, kk, false)};
    const bool filled = beside > 0;
    static const struct {
        int cfg;
        TileTime t;
    } menu[] = {{GEMM_WIDE, {3.0, 0.90, false}},
                {GEMM_SPLIT, {2.4, 0.47, false}},
                {GEMM_MID, {2.0, 0.50, false}},
                {GEMM_FLAT, {1.0, 0.42, true}},
                {GEMM_SMALL, {1.0, 0.27, true}}};
    GemmChoice best{GEMM_FEW, -1.0};
    const int64_t few = gemm_tiles(GEMM_FEW, m, n);
    if (few <= 512)  // (two on a compute unit: where a wave's share is one step the second costs 0.6 of the first)
        best.us = 2.5 + (few <= 256 ? 1.0 : kk <= kFewSingle ? 1.6 : 2.0) * (1.0 + 0.85 * (double)kk / (double)kFewSingle);
    for (const auto &e : menu) {
        const double us = tile_us(e.t, gemm_tiles(e.cfg, m, n), kk, filled);
        if (best.us < 0.0 || us < best.us) best = GemmChoice{e.cfg, us};
    }
    return best;
}
// The tile of a product: with no other work-groups in its launch, a second look by times of the tiles as they are, for what they call 4 % and
// half a microsecond.  A step takes longer the more of the compute units run one (`full`); of the small tiles two share one, a full round of which takes `two` times, one of
// 257 and more from `over` times on.  Fitted to 2800 products (1 to 16384 rows, 256 to 4096 columns, contractions from 16 to 4096; Y, dX and
// dW alike): 1480 of more than 6.5 us: the tile that choose_gemm takes is 4.4 % slower than the fastest on average and 68 % at most, this one 0.4 %,
// and 1.06 of the time before at most.  What it mends most is few_tile, whose chain of loads is longer than that of 64 x 64 tiles where a wave has
// several steps (dW 1088 x 272, k = 1407: 12.7 -> 8.0 us; Y 124 x 2496 -> 2496 11.9 -> 9.4), and 64 x 64 tiles in 257 to 400 work-groups (dW 280
// x 3496, k = 1805: 17.6 -> 13.5 on 64 x 128).
inline double gemm_us(int cfg, int64_t m, int64_t n, int64_t kk) {
    static const struct {
        double launch, fix, step, full, over, two;  // (`over` 0: a compute unit each)
    } times[] = {{0.95, 5.42, 0.804, 1.01, 0.0, 0.0}, {1.41, 3.55, 0.441, 0.93, 0.0, 0.0}, {2.23, 2.61, 0.247, 1.18, 0.0, 0.0}, {2.59, 1.85, 0.259, 1.07, 0.0, 0.0},
                 {3.41, 0.76, 0.163, 1.37, 1.48, 1.77}, {3.29, 0.72, 0.123, 1.04, 1.51, 1.70}, {3.53, 0.00, 0.682, 0.74, 1.54, 1.87}};  // (in the order of GEMM_LARGE ..)
    const auto &t = times[cfg];
    const int64_t tiles = gemm_tiles(cfg, m, n), rest = tiles % 512;
    const double rounds = t.over == 0.0 ? (double)((tiles + 255) / 256)
                                        : t.two * (double)(tiles / 512) + (rest == 0 ? 0.0 : rest <= 256 ? 1.0 : t.over + (t.two - t.over) * (double)(rest - 256) / 256.0);
    const int64_t steps = cfg == GEMM_FEW ? ((kk + 15) / 16 + 31) / 32 : (kk + 63) / 64;  // (of a wave / of the work-group)
    return t.launch + rounds * (t.fix + t.step * (double)steps * (1.0 + t.full * (tiles < 256 ? (double)tiles / 256.0 : 1.0)));
}
inline int gemm_cfg(int64_t m, int64_t n, int64_t kk, int64_t beside = 0) {
    const int first = choose_gemm(m, n, kk, beside).cfg;
    if (beside > 0) return first;
    int best = first;
    double best_us = 0.96 * gemm_us(first, m, n, kk) - 0.5;
    if (best_us < 4.2) return first;  // (no tile takes less than 4.13: nothing to gain)
    for (int cfg = gemm_tiles(GEMM_LARGE, m, n) >= 130 ? GEMM_LARGE : GEMM_WIDE; cfg <= GEMM_FEW; ++cfg) {
        if (cfg == GEMM_FEW && gemm_tiles(GEMM_FEW, m, n) > 512) continue;
        const double us = gemm_us(cfg, m, n, kk);
        if (us < best_us) best = cfg, best_us = us;
    }
    return best;
}

// |X^T dY|_F^2 per tile for the variance monitors: the dW-type product (both operands stored
// [token][feature]) with the squared-norm epilogue; the tiles of the other products, but for 32 x 32, beside the work-groups of
// the row norms (6670 tokens, 608 x 1704: 270 tiles of 64 x 64 63 us, 140 of 64 x 128 49).
// Where 128 x 128 tiles take nearly all compute units and are short, the row norms that find none free are a round of their own; there two
// work-groups to a compute unit (524 tokens, 2824 x 1312: 253 tiles and 66 work-groups of norms 15.4 us, so 12.8; fourteen such shapes of 261
// to 1594 tokens 0.79 to 0.98 of the time.  Of 2412 tokens and more 0.96 to 1.46, of fewer tiles 0.87 to 1.46, most of them above 1).
// In scratch for less than a partial sum of each of these, 128 x 128 tiles.
inline int xty_cfg(int64_t m, int64_t n, int64_t kk, int64_t room = INT64_MAX) {
    const int cfg = gemm_cfg(m, n, kk, row_norm_blocks(kk)), small = cfg == GEMM_FEW ? GEMM_SMALL : cfg;
    const int64_t mid = gemm_tiles(GEMM_MID, m, n);
    if ((small == GEMM_MID || small == GEMM_SPLIT) && mid >= 216 && mid <= 256 && mid + row_norm_blocks(kk) > 256 && kk >= 256 && kk <= 2048 &&
        mid <= room)
        return GEMM_COMPACT;
    return gemm_tiles(small, m, n) <= room ? small : kk >= 1536 ? GEMM_SPLIT : GEMM_MID;
}
inline int xty_sumsq_tiles(int64_t n, int64_t d_in, int64_t d_out, int64_t room = INT64_MAX) {
    return (int)gemm_tiles(xty_cfg(d_in, d_out, n, room), d_in, d_out);
}

// Which kernel serves a sketch product (with k > kSmallK, or fewer columns in a paired launch) and how its token dimension is cut.  The work-group
// generates the sketch tile into LDS and all eight waves read it.
struct SketchPlan {
    int cfg;
    int slices, per_tail;  // slices of k_chunk tokens of every tile; tiles per work-group that takes short last slices (0: there are none)
    int splits;            // slices of a tile, the short one included
    int64_t k_chunk, tiles;
    int shares() const { return slices * (int)tiles + (per_tail > 0 ? (int)((tiles + per_tail - 1) / per_tail) : 0); }
};

// Tokens are cut into slices of `k_chunk` tokens (a multiple of 64) so that about `target_wgs` work-groups exist
// (256 = one per compute unit; measured: more or fewer are slower when the product runs alone); with more than
// one slice the kernel writes fp32 partial results to workspace and reduce_partials_kernel sums them in slice
// order.  104 tiles would get two slices each, and 48 compute units nothing to do.  So a tile may also get a last,
// shorter slice; the work-groups left over take those of per_tail tiles each, as long in all as a long slice
// (16384 x 4096, k = 1638: 111 steps on 243 compute units instead of 128 on 208, with the sum of the slices 253 ->
// 235 us, Rademacher 208 -> 194; k = 819 129 -> 130 and 110 -> 107).
// `overhead` is what a tile costs besides its steps, in steps; a tile gets at most `most` slices.
inline void slice_sketch(SketchPlan &p, int64_t n, int target_wgs, double overhead, int64_t most) {
    const int64_t units = (n + 63) / 64;
    int64_t s = target_wgs / p.tiles;
    if (s > (units + 1) / 2) s = (units + 1) / 2;  // (a slice of one step: 1000 x 2000, k = 100 12.9 -> 14.7 us)
    if (s > most) s = most;
    if (s < 1) s = 1;
    int64_t len = (units + s - 1) / s;
    p.slices = p.splits = (int)((units + len - 1) / len), p.per_tail = 0;
    const int64_t spare = target_wgs - s * p.tiles;
    if (spare > 0 && s < most) {
        const int64_t m = (p.tiles + spare - 1) / spare;
        const double tail = ((double)units + overhead) * (double)m / (double)(s * m + 1);
        const int64_t tail_len = (int64_t)tail + ((double)(int64_t)tail < tail ? 1 : 0);
        if (s * tail_len < units && (double)tail_len < 0.92 * (double)len)
            len = tail_len, p.slices = (int)s, p.splits = (int)s + 1, p.per_tail = (int)m;
    }
    p.k_chunk = len * 64;
}

// The tiles of a sketch product, and the time of a 64-token step on a full chip (alone).
struct SketchMenu {
    int64_t bm, bn;
    double step_us[2];  // Gaussian, Rademacher
};
constexpr int kSketchTiles = 6;
constexpr SketchMenu kSketchMenu[kSketchTiles] = {{128, 256, {1.18, 0.91}}, {128, 512, {1.92, 1.63}}, {64, 512, {1.20, 1.04}},  // (in the order of SK_NARROW ..)
                                                  {64, 384, {0.93, 0.86}},  {128, 384, {1.54, 1.30}}, {64, 256, {0.85, 0.61}}};

// The tile is the one of the menu whose time comes out lowest: rounds of 256 work-groups, each as long as
// its slice's 64-token steps, plus the partial results.  The times of a step on a full chip come from a fit over
// measured shapes, adjusted by hand where another choice was faster; partial results cost 0.2 us per MB written and
// read (they mostly stay in the last-level cache).  What that weighs: padding of k and d, entries generated once per
// 512, 384 or 256 columns, operand columns staged once per 128 or 64 rows, and filling the chip when tokens are few.
// It ranks the tiles and does not predict: what every tile costs alike (launch, first step, 8 us and more at small
// sizes) is left out.  All six tiles timed at sixteen shapes from 2000 x 400, k = 100 to 16384 x 4096, k = 1638
// (profiles/sketch_products.txt): the one taken is 2.0 % slower than the fastest on average with the Gaussian kind,
// 18 % at most (32000 x 512, k = 640: 49 us, 128 x 256 42), 0.3 and 1.9 % with Rademacher.  ((16384 x 4096, k = 410)
// 64 x 512: 79 us, 128 x 512: 107; (10000 x 3000, k = 1000) 128 x 384: 81, 64 x 256: 108; 4096 x 3072, k = 3686
// unsliced on 128 x 384: 102, 128 x 512: 107.)
// `limited`: the caller may be rmm_sketch_static.  `room`: token slices that the caller's scratch holds.
constexpr int64_t kMostSlices = 64;
inline int64_t most_static_slices(int64_t n, int64_t d, int64_t k) {
    // rmm_sketch_static serves the shapes whose partial results fit RMM_STATIC_SCRATCH_BYTES with the plainest
    // tiling (rows by k, columns by d); those keep fitting, whichever tile they run with.
    const int64_t fit = (int64_t)((double)RMM_STATIC_SCRATCH_BYTES / ((double)k * (double)d * 4.0));
    if (fit >= kMostSlices) return kMostSlices;
    const int64_t tiles = d >= 1024 ? tiles_of(k, d, k <= 512 ? 64 : 128, 512) : d % 384 == 0 ? tiles_of(k, d, k <= 512 ? 64 : 128, 384) : tiles_of(k, d, 128, 256);
    const int64_t blocks = (n + 127) / 128, s = tiles >= 256 ? 1 : blocks < 256 / tiles ? blocks : 256 / tiles;
    const int64_t chunk = (blocks + s - 1) / s, slices = (blocks + chunk - 1) / chunk;
    return slices == 1 || slices <= fit ? (fit < 1 ? 1 : fit) : kMostSlices;
}
inline SketchPlan plan_sketch_in(int64_t n, int64_t d, int64_t k, int kind, int64_t most) {
    SketchPlan best{};
    double best_us = -1.0;
    static const int order[kSketchTiles] = {SK_WIDE64, SK_WIDE, SK_MID64, SK_MID, SK_NARROW64, SK_NARROW};
    for (int cfg : order) {
        const SketchMenu &e = kSketchMenu[cfg];
        SketchPlan p;
        p.cfg = cfg, p.tiles = tiles_of(k, d, e.bm, e.bn);
        const double step_us = e.step_us[kind != 0];
        if (best_us >= 0.0 && (double)p.tiles * (double)((n + 63) / 64) * step_us >= 256.0 * best_us) continue;  // (its steps alone, on a full chip)
        slice_sketch(p, n, 256, 4.0 / step_us, most);
        const double us = (double)((p.shares() + 255) / 256) * (double)(p.k_chunk / 64) * step_us + 2.0 * p.per_tail +
                          (p.splits > 1 ? (double)p.splits * (double)k * (double)d * 0.82e-6 : 0.0);
        if (best_us < 0.0 || us < 0.98 * best_us) best = p, best_us = us;  // (ties: the wider tile)
    }
    return best;
}
inline SketchPlan plan_sketch(int64_t n, int64_t d, int64_t k, int kind, bool limited, int64_t room = kMostSlices) {
    const int64_t most = limited ? most_static_slices(n, d, k) : kMostSlices;
    return plan_sketch_in(n, d, k, kind, room < most ? room : most);
}

// The streaming kernel of small sketch sizes: token slices so that about one work-group per
// compute unit exists; 2 register sets of loads in flight.  Work-groups take 256 columns, or 128
// where that would leave slices of at most 2048 tokens (k <= 32) / 512 tokens (k <= 64): half as many,
// twice as long slices then halve the partial sums and the final cross-wave sum of a work-group
// (measured: 26.6 against 27.6 us at 16384 x 4096, k = 32; 11.7 against 15.3 us at 16384 x 1024),
// while on long slices the wider work-group is ahead (82.8 against 84.6 us at 65536 x 4096).
constexpr int64_t kSmallK = 64;
inline int smallk_slices_for(int64_t n, int64_t d, int64_t bn, int64_t *k_chunk) {
    const int64_t col_tiles = (d + bn - 1) / bn, blocks = (n + 127) / 128;
    int64_t s = 256 / col_tiles;
    if (s > blocks) s = blocks;
    if (s < 1) s = 1;
    *k_chunk = (blocks + s - 1) / s * 128;
    return (int)((n + *k_chunk - 1) / *k_chunk);
}
inline int64_t smallk_bn(int64_t n, int64_t d, int64_t k) {
    int64_t k_chunk;
    (void)smallk_slices_for(n, d, 256, &k_chunk);
    return k_chunk <= (k <= 32 ? 2048 : 512) ? 128 : 256;
}
inline int smallk_slices(int64_t n, int64_t d, int64_t k, int64_t *k_chunk) {
    return smallk_slices_for(n, d, smallk_bn(n, d, k), k_chunk);
}

// ---- Paired launches: which tiles and slices a pass takes.

// Time until `second` jobs of t2 us each are done that follow `first` jobs of t1 us on `slots` equal slots (256 or 512).
inline double makespan(int64_t first, double t1, int64_t second, double t2, int64_t slots) {
    const int64_t late = first & (slots - 1), early = slots - late;  // slots that become free a round later / at once
    const double base = (double)(slots == 512 ? first >> 9 : first >> 8) * t1;
    double t = 0.0;
    for (int64_t i = 0, j = 0, done = 0; done < second;) {  // rounds of the early slots and of the late ones, by the time they end
        const double e = (double)(i + 1) * t2, l = late > 0 ? t1 + (double)(j + 1) * t2 : 1e30;
        if (e <= l)
            t = e, ++i, done += early;
        else
            t = l, ++j, done += late;
    }
    return base + (late > 0 && t < t1 ? t1 : t);
}

// us of a work-group of either product of a paired launch, what share of that (`full`) all of them take longer on a full chip, and how many run at a
// time.  Plans are compared by the hundred for every size that is new, so those are not walked through whose work, shared evenly by all slots, or one of whose
// work-groups takes as long as the best plan so far (workspace queries of both directions of 768 <-> 3072 at 3600 to 8000 tokens, four plans: 30 us when all
// were walked through, 10 now, 4 of them without the second look; k = 32 16 and 8).
struct PairTimes {
    double plain, sketch, full_plain, full_sketch;
    int64_t slots;
    double full(int64_t tiles, int64_t shares) const { return (full_plain * (double)tiles * plain + full_sketch * (double)shares * sketch) / (double)slots; }
    double work(int64_t tiles, int64_t shares) const { return ((double)tiles * plain + (double)shares * sketch) / (double)slots; }
    double least(int64_t tiles, int64_t shares) const {
        const double even = work(tiles, shares), one = plain > sketch ? plain : sketch;
        return even > one ? even : one;
    }
};

// us of a paired launch and the sum of its slices: work-groups of either kind take a time of their own (first loads and
// writing, and every step of 64 contraction elements) and are dealt to 256 slots in grid order, or to 512 where two share
// a compute unit.  The times are fitted to 4300 launches of 60 passes (256 to 16384 tokens, widths 256 to 4096,
// k = 73 to 6911; all sketch tiles, 64 to 512 work-groups): 7 % rms off.  Over those passes the plan it leads to is 3.3 % slower than the
// best one on average and 30 % at most; plans made for the sketch product alone were 12 and 50 %.  (As above: from before the loops.)
inline PairTimes pair_times(const PairPlain &plain, int64_t kk, const SketchPlan &p, int kind, bool limited) {
    struct Times {
        double fix, step;
    };
    static const Times large{6.3, 1.405}, mid{3.4, 0.487}, mid_long{4.0, 0.478}, compact{5.4, 0.733};  // (mid_long: contractions from 1536 on)
    struct SketchTimes {
        double fix, step[2];  // Gaussian, Rademacher
    };
    static const SketchTimes sk_compact{5.5, {1.009, 0.935}}, sk_compact_two{5.5, {1.28, 1.07}};
    static const SketchTimes sk[] = {{5.3, {1.288, 0.957}}, {7.2, {1.651, 1.476}}, {5.1, {1.078, 1.080}},   // (in the order of SK_NARROW ..)
                                     {5.0, {0.929, 0.910}}, {6.3, {1.490, 1.192}}, {4.05, {0.780, 0.722}}};
    const bool two = plain.cfg == GEMM_COMPACT;
    const Times &a = plain.cfg == GEMM_LARGE ? large : two ? compact : kk >= 1536 ? mid_long : mid;
    // sk_compact_two: unsliced sketch work-groups that come first and are more than the compute units share some for all of their
    // time (87 launches; 4859 x 1928 -> 520, k = 2430, 304 of them: 118 us where 82 were planned, another plan 90).  `limited` plans, which
    // say the least scratch of a pass, are made without.
    const SketchTimes &b = !two ? sk[p.cfg] : !limited && p.slices == 1 && p.shares() > 256 ? sk_compact_two : sk_compact;
    const double ta = a.fix + a.step * (double)((kk + 63) / 64), tb = b.fix + b.step[kind != 0] * (double)(p.k_chunk / 64);
    return PairTimes{ta, tb, 0.0, 0.0, two ? 512 : 256};
}
// (`enough`: a plan that cannot be below need not be told exactly)
inline double pair_us(const PairPlain &plain, int64_t kk, const SketchPlan &p, int kind, double partial_mb, bool limited = false, double enough = 1e30) {
    const PairTimes us = pair_times(plain, kk, p, kind, limited);
    const double ta = us.plain, tb = us.sketch, sum = p.splits > 1 ? 2.6 + 0.213 * (double)p.splits * partial_mb : 0.0;
    if (const double least = us.least(plain.tiles, p.shares()) + sum; least >= enough) return least;
    double t = sketch_goes_first(plain.tiles, p.slices) ? makespan(p.shares(), tb, plain.tiles, ta, us.slots)
                                                        : makespan(plain.tiles, ta, p.shares(), tb, us.slots);
    // Beside 256 x 256 tiles, several rounds of them, power limits the chip's clock and a sketch work-group as long as the launch takes a
    // tenth more (16384 x 1024 -> 4096, k = 1638, Rademacher: 78 work-groups of 169 us by the times above 202 us with the sum of the
    // slices, 91 of 115 185).
    if (plain.cfg == GEMM_LARGE && plain.tiles > 256 && t < 1.1 * tb) t = 1.1 * tb;
    return t + sum;
}

// Of at most kSmallK columns a pass takes no more slices than this: a quarter more than the streaming kernel of the product alone, and one.
inline int64_t most_slices_of_pass(int64_t n, int64_t d_sk, int64_t k, int64_t room) {
    if (k > kSmallK) return room;
    int64_t k_chunk;
    const int64_t alone = smallk_slices(n, d_sk, k, &k_chunk), most = alone + alone / 4 + 1;
    return room < most ? room : most;
}

struct PassPlan {
    PairPlain plain;
    SketchPlan sketch;
    bool sketch_first;  // the sketch work-groups stand in front of the plain tiles
};

// us of a pass by times of the tiles as they are: work-groups as in pair_us, and the sum of the slices.  The fuller the chip, the longer all of them
// take (`full`: power, and lines from L2).  What a round more or less would change is taken at plain tiles of 0.9 and of 1.1 of their time
// (`plain_times`), so that no plan is taken for a round that it may just miss.  Fitted to 135000 launches of 446 passes with kSecondLookProducts and more (all sketch tiles, 64 to 512
// work-groups of them, either order).
inline PairTimes pass_times(const PassPlan &p, int64_t kk, int kind) {
    struct Times {
        double fix, step, full;
    };
    static const Times large{4.56, 0.844, 0.63}, wide{1.67, 0.537, 0.66}, mid{1.20, 0.426, 0.46}, compact{2.30, 0.673, 0.66};
    struct SketchTimes {
        double fix, step[2], full;  // Gaussian, Rademacher
    };
    static const SketchTimes sk_compact{3.05, {0.818, 0.725}, 0.31};
    static const SketchTimes sk[] = {{3.18, {0.909, 0.763}, 0.36}, {4.88, {1.096, 1.062}, 0.36}, {2.81, {0.784, 0.997}, 0.43},   // (in the order of SK_NARROW ..)
                                     {3.51, {0.699, 0.874}, 0.37}, {5.14, {0.990, 0.965}, 0.37}, {2.66, {0.589, 0.573}, 0.31}};
    const bool two = p.plain.cfg == GEMM_COMPACT;
    const Times &a = p.plain.cfg == GEMM_LARGE ? large : p.plain.cfg == GEMM_WIDE ? wide : two ? compact : mid;
    const SketchTimes &b = two ? sk_compact : sk[p.sketch.cfg];
    const double ta = a.fix + a.step * (double)((kk + 63) / 64), tb = b.fix + b.step[kind != 0] * (double)(p.sketch.k_chunk / 64);
    return PairTimes{ta, tb, a.full, b.full, two ? 512 : 256};
}
inline double pass_sum_us(const SketchPlan &p, double partial_mb) { return p.splits > 1 ? 1.2 + 0.304 * (double)p.splits * partial_mb : 0.0; }
inline double pass_us(const PassPlan &p, int64_t kk, int kind, double partial_mb, std::initializer_list<double> plain_times = {0.89, 1.11}) {
    const PairTimes us = pass_times(p, kk, kind);
    const int64_t tiles = p.plain.tiles, shares = p.sketch.shares();
    double longest = 0.0;
    for (double f : plain_times)
        longest += p.sketch_first ? makespan(shares, us.sketch, tiles, f * us.plain, us.slots) : makespan(tiles, f * us.plain, shares, us.sketch, us.slots);
    return longest / (double)plain_times.size() + us.full(tiles, shares) + pass_sum_us(p.sketch, partial_mb);
}

// The plain product of a pass (n x m outputs) beside a sketch product on one work-group per compute unit: 256 x 256 tiles where it
// fills the chip with them, else 128 x 128.  ShapeCompact adds in the order of ShapeMid, so that the bits of Y follow from its
// sizes alone, whatever the sketch is.
inline PairPlain pair_plain(int64_t n, int64_t m) {
    const int cfg = gemm_tiles(GEMM_LARGE, n, m) >= 160 ? GEMM_LARGE : GEMM_MID;
    return PairPlain{cfg, (int)gemm_tiles(cfg, n, m)};
}
// dX with a long contraction runs with two wave groups on these tiles: its row-indexed operand is read from LDS half as often
// (backward, 2048 x 1024 -> 4096, k = 205: 36.5 us, without 38.7; Y gains nothing: over 49 passes with contractions from 1536 on
// 0.994 of the time without them).
inline int dx_cfg(int cfg, int64_t kk) { return cfg == GEMM_MID && kk >= 1536 ? GEMM_SPLIT : cfg; }

// More token slices than a pass may have over its sketch product alone.
inline bool too_many(int splits, int of_alone) { return splits > 1 && (of_alone == 1 || 4 * (splits - 1) > 5 * of_alone); }

// The sketch product of a pass by itself.
struct SketchAlone {
    SketchPlan plan;  // as rmm_sketch_static has it
    int free_splits;  // slices without that limit
};
inline SketchAlone sketch_alone(int64_t n, int64_t d, int64_t k, int kind, bool limited, int64_t room) {
    const int64_t most = most_static_slices(n, d, k);
    const SketchPlan p = plan_sketch_in(n, d, k, kind, room < most ? room : most);
    return SketchAlone{p, limited || room <= most ? p.splits : plan_sketch_in(n, d, k, kind, room < kMostSlices ? room : kMostSlices).splits};
}

// Plan of a pass: sketch of the n x d_sk operand, plain product n x d_other over d_sk.  Every sketch tile with slices for 64
// to 320 work-groups, and 64 x 256 tiles with ShapeCompact where all work-groups are resident at once.  (4096 x 768 ->
// 768, k = 410, with the sum of its slices: 26.9 -> 21.3 us; 4096 x 3072 -> 768, k = 2048, Rademacher 82 -> 69; 3001 x 1304 ->
// 520, k = 600: 32 -> 24.)  At most a quarter more slices than alone, and one more (two may become three; where the product
// alone has one the pass has one): by so much a pass may ask for more scratch than its sketch product.  (Without the one, 3 % of the
// passes of those ranges take other plans, 4 % slower on average; the worst of 60: 13986 x 376 -> 1808, k = 6993, Rademacher,
// forward 102 -> 132 us.)  Less than 0.8 us, which is what the model is off by at the smallest sizes, is not worth another order of additions
// than that of the product alone.
// The product alone is taken as rmm_sketch_static has it, whose partial sums are few.  A pass may have more of them, by as much over what
// the product alone takes without that limit, for 8 % of the model's time (`limited`: not so).  (12531 x 760 -> 272, k =
// 6265, Rademacher, forward: 172 us in one slice, 124 in two and a short one; 26 of 260 passes with k from a fifth of the tokens on, 8 % faster
// on average, 1.00 to 1.20.  With a margin of 5 % two of 28 lose 5 %.)
constexpr int kCutTargets[] = {64, 96, 128, 160, 192, 224, 256, 320, 384, 448, 512};
constexpr int kCuts = sizeof(kCutTargets) / sizeof(int);
// The ways to cut a sketch product, each made when it is first asked for.
class SketchCuts {
public:
    SketchCuts(int64_t n, int64_t d_sk, int64_t k, int kind, int64_t room) : n_(n), room_(room), kind_(kind != 0) {
        for (int cfg = 0; cfg < kSketchTiles; ++cfg) {
            for (SketchPlan &p : plans_[cfg]) p.slices = 0;
            tiles_[cfg] = tiles_of(k, d_sk, kSketchMenu[cfg].bm, kSketchMenu[cfg].bn);
        }
    }
    const SketchPlan &get(int cfg, int target) {
        SketchPlan &p = plans_[cfg][target];
        if (p.slices == 0) {
            p.cfg = cfg, p.tiles = tiles_[cfg];
            slice_sketch(p, n_, kCutTargets[target], 4.0 / kSketchMenu[cfg].step_us[kind_], room_);
        }
        return p;
    }
    // on tiles of `cfg` in one slice: no slices of it are less work
    SketchPlan whole(int cfg) const { return SketchPlan{cfg, 1, 0, 1, (n_ + 63) / 64 * 64, tiles_[cfg]}; }

private:
    int64_t n_, room_, tiles_[kSketchTiles];
    int kind_;
    SketchPlan plans_[kSketchTiles][kCuts];  // (slices = 0: not cut yet)
};
inline PassPlan first_plan(SketchCuts &cuts, int64_t n, int64_t d_sk, int64_t d_other, int64_t k, int kind, bool limited, const SketchAlone &alone) {
    const double partial_mb = (double)k * (double)d_sk * 4e-6;
    const PairPlain usual = pair_plain(n, d_other);
    const PairPlain compact{GEMM_COMPACT, (int)gemm_tiles(GEMM_COMPACT, n, d_other)};
    PassPlan best{usual, alone.plan, false};
    double best_us = pair_us(usual, d_sk, alone.plan, kind, partial_mb, limited) - 0.8;
    for (int cfg = 0; cfg < kSketchTiles; ++cfg) {
        const SketchPlan whole = cuts.whole(cfg);
        const bool may_share = cfg == SK_NARROW64 && usual.cfg != GEMM_LARGE && compact.tiles + whole.tiles <= 512;
        if (!may_share && pair_times(usual, d_sk, whole, kind, limited).work(usual.tiles, whole.tiles) >= best_us) continue;
        int slices = -1, per_tail = -1;
        for (int target : {0, 1, 2, 4, 6, 7}) {
            const SketchPlan &p = cuts.get(cfg, target);
            if (p.slices == slices && p.per_tail == per_tail) continue;
            slices = p.slices, per_tail = p.per_tail;
            const bool many = too_many(p.splits, alone.plan.splits);
            if (many && too_many(p.splits, alone.free_splits)) continue;
            const double worth = many ? 1.08 : 1.0;
            double us = worth * pair_us(usual, d_sk, p, kind, partial_mb, limited, 1.0001 * best_us / worth);
            if (us < best_us) best = PassPlan{usual, p, false}, best_us = us;
            if (!may_share || compact.tiles + p.shares() > 512) continue;
            us = worth * pair_us(compact, d_sk, p, kind, partial_mb, limited, 1.0001 * best_us / worth);
            if (us < best_us) best = PassPlan{compact, p, false}, best_us = us;
        }
    }
    best.sketch_first = sketch_goes_first(best.plain.tiles, best.sketch.slices);
    return best;
}

// What a pass asks for three times (workspace of either kind, launch) and depends on its sizes alone, remembered by each thread.  In sets
// of four places, the latest first, so that the four plans of a layer, both kinds and directions, never put each other out.  (In single places the
// directions of one in 64 layers of few sketch columns did, in pairs three of the four plans of one in 260: its queries took 7 us and more, 50 ns each now.)
struct Sizes {
    int64_t n, d_sk, d_other, k, what;
    bool operator==(const Sizes &o) const { return n == o.n && d_sk == o.d_sk && d_other == o.d_other && k == o.k && what == o.what; }
};
template <typename Value, typename Make>
Value remembered(const Sizes &s, Make make) {
    struct Entry {
        Sizes sizes;
        Value value;
    };
    constexpr size_t SETS = 32, PLACES = 4;
    static thread_local Entry memo[SETS][PLACES];  // (n = 0: empty)
    const uint64_t h = ((uint64_t)s.n * 0x9E3779B97F4A7C15u ^ (uint64_t)s.d_sk * 0xC2B2AE3D27D4EB4Fu ^ (uint64_t)s.d_other * 0x165667B19E3779F9u ^
                        (uint64_t)s.k * 0x27D4EB2F165667C5u) + (uint64_t)s.what * 0xD6E8FEB86659FD93u;
    Entry *set = memo[(h ^ h >> 32) % SETS];
    for (size_t i = 0; i < PLACES; ++i)
        if (set[i].sizes == s) return set[i].value;
    const Entry made{s, make()};
    for (size_t i = PLACES - 1; i > 0; --i) set[i] = set[i - 1];  // (the oldest goes)
    return (set[0] = made).value;
}

// Passes of at most kSmallK sketch columns: the paired launch, or the product and the streaming kernel one after the other.  The latter
// computes no more rows than k asks for, where a sketch tile has 64 at least; but it reads A a second time by itself, in at most 256
// work-groups that each go through their tokens alone (2.3 us per 64 of them, or 5 us and 5 TB/s where that is less), and ends with the sum of
// its slices (0.4 us each), and beside the product's tiles the padding costs less than that.  Taken where the fitted time of the pair is 5 % less
// than that of the two.  Over 1510 passes that were timed both ways (40 to 250000 tokens, widths 64 to 4096, k = 1 to 64) it takes 0.86 of the
// time on average, as the better of the two each time does (forward 4224 x 848 -> 560, k = 64: 27.2 -> 16.0 us; 738 x 384 -> 2656: 13.3 ->
// 8.7), and in 9 of them more than 1.025, 1.07 at most.  Without the 5 TB/s 1.34 at most (3982 x 3760 -> 200, k = 13: 29.9 -> 40.1); always in
// pairs: up to 1.8 where few rows meet long contractions, for which gemm_cfg has tiles that a pair has not.  Work-groups that are not all resident at once
// do not read the same of A at the same time: a pair of more than a round is no shorter than A twice at 3.6 TB/s (750 others, most of them long operands beside
// few columns of Y or dX: 0.829 of the time and 25 above 1.025 without that, 1.18 at most (dY of 51799 x 1984 with dX 144 wide, k = 11: 84 -> 98 us); 0.833
// and 7 with it, 1.10 at most; 500 fresh ones of all sizes 0.806, 9 above 1.025, three of them above 1.1: 1286 x 1328 -> 640, k = 1, forward 14.0 -> 17.4, 25203 x
// 2656 -> 808, k = 3, 152 -> 173, dX of 182443 x 1224 with dX 384 wide, k = 1, 303 -> 335).  Asked of the plan that the second look below starts from: it takes another one only where that is much shorter.
struct SmallPass {
    bool paired;
    PassPlan first;  // of the Gaussian kind, which answers for either
};
inline SmallPass small_pass(int64_t n, int64_t d_sk, int64_t d_other, int64_t k) {
    return remembered<SmallPass>(Sizes{n, d_sk, d_other, k, 0}, [&] {
        int64_t k_chunk;
        const int slices = smallk_slices(n, d_sk, k, &k_chunk);
        const double steps_us = 2.3 * (double)(k_chunk / 64), read_us = 5.0 + (double)n * (double)d_sk * 2e-6 / 5.0;
        const double apart = 1.1 * gemm_us(gemm_cfg(n, d_other, d_sk), n, d_other, d_sk) + (steps_us < read_us ? steps_us : read_us) + 0.4 * (double)slices;
        const int64_t room = most_slices_of_pass(n, d_sk, k, kMostSlices);
        SketchCuts cuts(n, d_sk, k, 0, room);
        const PassPlan pass = first_plan(cuts, n, d_sk, d_other, k, 0, false, sketch_alone(n, d_sk, k, 0, false, room));
        double pair = pair_us(pass.plain, d_sk, pass.sketch, 0, (double)k * (double)d_sk * 4e-6);
        const double twice = 2.0 * (double)n * (double)d_sk * 2e-6 / 3.6;
        if (pass.plain.tiles + pass.sketch.shares() > (pass.plain.cfg == GEMM_COMPACT ? 512 : 256) && pair < twice) pair = twice;
        return SmallPass{pair * 1.05 + 0.5 < apart, pass};
    });
}
inline bool small_pass_is_paired(int64_t n, int64_t d_sk, int64_t d_other, int64_t k) { return k <= kSmallK && small_pass(n, d_sk, d_other, k).paired; }

// A second look at large passes, by pass_us: 256 x 256 tiles also where they do not fill the chip, 128 x 256 tiles, and either order, with any sketch
// tile.  At headline size dX on 96 tiles of 128 x 256 beside 112 sketch work-groups of 64 x 384, a compute unit each, takes the place
// of 192 tiles of 128 x 128 two by two with 168 of 64 x 256: a step that two work-groups of a compute unit share takes them 0.8 us, and some
// units have one, some two (a step 84.3 -> 75.8 us; 4096 x 3072 -> 768, k = 2048, Rademacher, two micro-batches: 310 -> 280; by box 1.09 to 1.11 and 1.085
// to 1.11 times as fast).
// Only for what the model calls 9 % or more, and 7 % with plain tiles of 1.2 of their time: on a full chip these slow down more than sketch
// work-groups do, and plans whose rounds of them just end with the sketch are not as short as the model has them.  Nor 256 x 256 tiles behind an
// unsliced sketch product that go over a round, which a chain of two or three such tiles ends (100 of them 0.80 to 1.26 of the time, a fifth above
// 1.025; 3078 x 928 -> 2960, k = 2631, forward: 51 -> 64 us).  It gives other plans to 45 % of the passes of these sizes: 421 of them were 0.895 of the time on
// average without these two rules, 18 above 1.025 and five above 1.1 (1180 x 2232 -> 2328, k = 1062, Rademacher, forward: 31 -> 35 us); 600 fresh ones are 0.894 with
// them, 18 above 1.025 and two above 1.1, 1.114 at most.  Of more than 8192 tokens 134 others are 0.99 on average and 7 of
// them 1.04 to 1.16: long launches, which slow the clock in a way that it does not know.  Below 6e9 products, 6 us of the matrix pipes, a pass is
// made up as much of launches, first loads and sums, and first_plan is 1 to 3 % behind the best plan.
constexpr double kSecondLookProducts = 6e9;
constexpr int64_t kSecondLookTokens = 8192;
inline PassPlan second_plan(const PassPlan &best, SketchCuts &cuts, int64_t n, int64_t d_sk, int64_t d_other, int64_t k, int kind, const SketchAlone &alone) {
    const double partial_mb = (double)k * (double)d_sk * 4e-6;
    PassPlan now = best;
    double now_us = 0.91 * pass_us(best, d_sk, kind, partial_mb);
    const double slow_us = 0.93 * pass_us(best, d_sk, kind, partial_mb, {1.2});
    struct Cut {
        SketchPlan plan;
        double longest, work, more;  // of one of its work-groups; shared evenly by all compute units; what a full chip and the sum of the slices add
    } some[kSketchTiles][kCuts];
    int count[kSketchTiles];  // (-1: not looked at yet)
    for (int &c : count) c = -1;
    for (int plain_cfg : {GEMM_LARGE, GEMM_WIDE, GEMM_MID}) {
        const PairPlain plain{plain_cfg, (int)gemm_tiles(plain_cfg, n, d_other)};
        for (int cfg = 0; cfg < kSketchTiles; ++cfg) {
            PassPlan p{plain, cuts.whole(cfg), false};
            const PairTimes us = pass_times(p, d_sk, kind);
            const double plain_work = us.work(plain.tiles, 0), plain_more = us.full(plain.tiles, 0);
            if (plain_work + plain_more + us.work(0, p.sketch.tiles) + us.full(0, p.sketch.tiles) >= 1.0001 * now_us) continue;  // (in one slice; more are no less)
            if (count[cfg] < 0) {
                count[cfg] = 0;
                int shares = -1;
                for (int target = 0; target < kCuts; ++target) {
                    p.sketch = cuts.get(cfg, target);
                    if (p.sketch.shares() == shares) continue;
                    shares = p.sketch.shares();
                    if (too_many(p.sketch.splits, alone.plan.splits) && too_many(p.sketch.splits, alone.free_splits)) continue;
                    const PairTimes t = pass_times(p, d_sk, kind);
                    some[cfg][count[cfg]++] = Cut{p.sketch, t.sketch, t.work(0, shares), t.full(0, shares) + pass_sum_us(p.sketch, partial_mb)};
                }
            }
            for (int i = 0; i < count[cfg]; ++i) {
                const Cut &c = some[cfg][i];
                double least = plain_work + c.work;
                if (least < us.plain) least = us.plain;
                if (least < c.longest) least = c.longest;
                if (least + plain_more + c.more >= 1.0001 * now_us) continue;
                p.sketch = c.plan;
                for (bool first : {false, true}) {
                    if (first && plain_cfg == GEMM_LARGE && c.plan.splits == 1 && plain.tiles + c.plan.shares() > 256) continue;  // (a chain of large tiles)
                    p.sketch_first = first;
                    const double all = pass_us(p, d_sk, kind, partial_mb);
                    if (all < now_us && pass_us(p, d_sk, kind, partial_mb, {1.2}) < slow_us) now = p, now_us = all;
                }
            }
        }
    }
    return now;
}
inline PassPlan make_pass_plan(int64_t n, int64_t d_sk, int64_t d_other, int64_t k, int kind, bool limited, int64_t room) {
    const bool known = k <= kSmallK && kind == 0 && !limited && room >= kMostSlices;  // (whether such a pass is paired has been asked before)
    room = most_slices_of_pass(n, d_sk, k, room);
    const bool again = !limited && n <= kSecondLookTokens && (double)n * (double)d_sk * (double)d_other >= kSecondLookProducts;
    if (known && !again) return small_pass(n, d_sk, d_other, k).first;
    const SketchAlone alone = sketch_alone(n, d_sk, k, kind, limited, room);
    SketchCuts cuts(n, d_sk, k, kind, room);
    const PassPlan best = known ? small_pass(n, d_sk, d_other, k).first : first_plan(cuts, n, d_sk, d_other, k, kind, limited, alone);
    return again ? second_plan(best, cuts, n, d_sk, d_other, k, kind, alone) : best;
}

// Plan of a pass, remembered.  With scratch for fewer slices than it takes, another one for these.
constexpr int64_t kLimited = -1;  // (in place of `room`: without a limit, the `limited` plan)
inline PassPlan plan_pass(int64_t n, int64_t d_sk, int64_t d_other, int64_t k, int kind, int64_t room = kMostSlices) {
    if (room >= kMostSlices) {
        room = kMostSlices;
    } else if (room != kLimited) {
        const PassPlan p = plan_pass(n, d_sk, d_other, k, kind);
        if (p.sketch.splits == 1 || p.sketch.splits <= room) return p;
    }
    kind = kind != 0;
    return remembered<PassPlan>(Sizes{n, d_sk, d_other, k, 2 * room + kind},
                                [&] { return make_pass_plan(n, d_sk, d_other, k, kind, room == kLimited, room == kLimited ? kMostSlices : room); });
}

// ---- The SORS kind: strips of eight columns of the sketched operand, which may share a launch with the plain product of their pass.

// Tokens as a power of two, 512 at least (the shortest transform of the strip kernel: 512 tokens of 768 columns on 1024 points take 5.8
// us instead of 5.4, of 4096 columns 6.9 instead of 6.1).  Up to 2048 a strip takes them in one piece, and
// any k; from there on in chunks of 2048, with accumulators for kSorsAccMaxK sketch columns, or kSorsManyK by twice the waves.
inline int sors_log(int64_t n) {
    int l = 9;
    while (((int64_t)1 << l) < n) ++l;
    return l;
}
constexpr int64_t kSorsAccMaxK = 2048;
// Work-groups of a strip beyond that, and the sketch columns of each, a multiple of four: one with kSorsManyK of them takes 1.45 times as long
// as one with next to none (16384 x 2048: 47.0 us and 33.6), and 256 of them run at a time.
constexpr int64_t kSorsManyK = 8192;
struct SorsParts {
    int64_t parts, part_k;
};
inline SorsParts sors_parts(int64_t d, int64_t k) {
    const int64_t need = (k + kSorsManyK - 1) / kSorsManyK;
    SorsParts best{};
    double best_time = -1.0;
    for (int64_t parts = need; parts < need + 8; ++parts) {
        const int64_t part_k = ((k + parts - 1) / parts + 3) / 4 * 4;
        const double time = (double)((d / 8 * parts + 255) / 256) * (1.0 + 0.45 * (double)part_k / (double)kSorsManyK);
        if (best_time < 0.0 || time < 0.99 * best_time) best = SorsParts{parts, part_k}, best_time = time;
    }
    return best;
}
inline int sors_chunks(int64_t n) { return sors_log(n) >= 12 ? 1 << (sors_log(n) - 11) : 1; }

enum { SORS_APART = 0, SORS_BEHIND = 1, SORS_FRONT = 2, SORS_COMPACT = 3 };
struct SorsPlan {
    int order;
    PairPlain plain;
};

// How a pass of n tokens launches the strips of a d_sk wide operand and its plain product, n x d_other over d_sk:
//   SORS_COMPACT  behind the tiles of ShapeCompact, one strip to a work-group: either needs half of a compute unit, so that the strips
//                 (vector units, LDS, memory) run beside tiles (matrix pipes) and fill places that these leave
//   SORS_BEHIND   two strips to a work-group, on the compute units that the last round of 256 x 256 or 128 x 128 tiles leaves, 32 or more
//   SORS_FRONT    the same in front of three or more rounds of tiles, on at most a quarter of the chip
//   SORS_APART    launches of their own
// The first by times fitted to 180 passes (513 to 16384 tokens, widths 256 to 4096).  Over 1517 others, 256 to 32768 tokens, passes
// take 0.890 of the time that they take with the others alone, dW included; 20 of them are more than 3 % longer, 1.17 at most; with
// hindsight 0.878.  (2275 x 312 -> 584, k = 455: a step 36.5 -> 25.5 us, 2907 x 1248 -> 1136 59.1 -> 44.5, 4250 x 1232 -> 864 71 -> 55.  Not where 256 x 256 tiles fill the chip, whose
// operands cost half the L2 traffic: 15053 x 2264 -> 3112 500 against 626; nor beside few tiles of a long contraction, which other
// tiles have more work-groups for: 3277 x 3480 -> 272 73 against 97.)  Of 100 passes of 1 to 512 tokens, widths
// 256 to 4096, it takes 20, which are 0.64 to 0.87 of the time that they were apart.
inline int sors_among_rounds(int64_t n, int64_t d_sk, int64_t d_other, int64_t k) {
    const PairPlain plain = pair_plain(n, d_other);
    if (sors_log(n) < 12 || sors_log(n) > 15 || k > kSorsAccMaxK) return SORS_APART;
    // (128 x 128 tiles: one round of them, long enough for the strips to finish beside it)
    if (plain.cfg != GEMM_LARGE && (plain.tiles < 65 || plain.tiles > 256 || d_sk < 768)) return SORS_APART;
    return (256 - plain.tiles % 256) % 256 >= 32 ? SORS_BEHIND : plain.tiles >= 256 && (d_sk / 8 + 1) / 2 <= 64 ? SORS_FRONT : SORS_APART;
}
inline SorsPlan plan_sors(int64_t n, int64_t d_sk, int64_t d_other, int64_t k) {
    const SorsPlan best{sors_among_rounds(n, d_sk, d_other, k), pair_plain(n, d_other)};
    const PairPlain &plain = best.plain;
    const int64_t l = sors_log(n), strips = d_sk / 8, pairs = (strips + 1) / 2;
    if (l > 15 || (l >= 12 && k > kSorsAccMaxK)) return best;
    const double steps = (double)((d_sk + 63) / 64), chunks = l < 11 ? 0.6 : (double)sors_chunks(n);
    const GemmChoice apart = choose_gemm(n, d_other, d_sk);
    double best_us;
    if (best.order != SORS_APART) {
        const double tile = plain.cfg == GEMM_LARGE ? 6.7 + 1.405 * steps : 3.4 + 0.487 * steps, two = 2.5 + 5.5 * chunks;
        best_us = 2.0 + (best.order == SORS_BEHIND ? makespan(plain.tiles, tile, pairs, two, 256) : makespan(pairs, two, plain.tiles, tile, 256));
    } else {
        best_us = apart.us + 5.4 + 2.2 * chunks * (strips <= 512 ? 1.0 : (double)strips / 512.0);
    }
    const PairPlain compact{GEMM_COMPACT, (int)gemm_tiles(GEMM_COMPACT, n, d_other)};
    const double strip = 3.8 + 2.5 * chunks, alone = 3.2 + 0.618 * steps, limit = (plain.cfg == GEMM_LARGE ? 0.9 : 1.0) * best_us;
    const SorsPlan shared{SORS_COMPACT, compact};
    if (compact.tiles + strips <= 256) return 2.5 + (alone > strip ? alone : strip) < limit ? shared : best;
    if (compact.tiles <= 256 && compact.tiles + strips <= 512) return 2.5 + alone + 0.41 * strip < limit ? shared : best;  // (some tiles start beside a strip)
    if (2.5 + makespan(compact.tiles, 3.8 + 0.836 * steps, strips, 3.8 + 3.9 * chunks, 512) >= limit) return best;
    // More work-groups than places: also by times taken since tiles of 256 columns have become faster than these, with two of these on a
    // compute unit told from one beside a strip (fitted to 311 forward passes that come here).  Of those and 260 backward passes 17 take more than 3 %
    // longer than with the others above, 1.17 of their time at most; without this second look 52, 1.32 at most (4187 x 3016 -> 2280, k = 419:
    // 113 and 86 us).  Of 500 passes that none of it was fitted to 4 take that
    // much longer than before there was a shared launch, 1.14 at most.  All 571 are 0.5 % shorter for it on average.
    const double two = compact.tiles <= 256 ? 0.0 : compact.tiles >= 512 ? 1.0 : (double)(compact.tiles - 256) / 256.0;
    const double now = 2.5 + makespan(compact.tiles, 3.5 + (0.832 + 0.279 * two) * steps, strips, 6.0 + 3.37 * chunks, 512);
    const double other = best.order != SORS_APART ? (plain.cfg == GEMM_LARGE ? 1.017 : 1.033) * best_us
                                                  : (apart.cfg == GEMM_LARGE ? 0.886 : apart.cfg == GEMM_WIDE ? 0.944 : 1.122) * apart.us + 4.2 +
                                                        (strips <= 256 ? 2.82 : 3.98 + 1.08 * (double)(strips - 256) / 256.0) * chunks;
    // (More than 16384 tokens, sixteen chunks, are beyond the passes that were fitted to, and tiles of many steps beside them take longer than
    // these times say: of 28 passes with contractions of 768 and more that came out below 0.97 and were taken, 16 were 1.04 to 1.16 of the time
    // (28837 x 824 -> 2968, k = 356, backward 253 us and 292); the 7 below 0.8 are 0.89 to 1.02.  41 with shorter contractions are 0.66 to 0.96.)
    const double margin = chunks > 8.0 && steps >= 12.0 ? 0.8 : apart.cfg == GEMM_LARGE ? 0.97 : 1.03;
    return now < margin * other ? shared : best;
}

// Whether the bias gradient's column sums go with dW: beside it where its launch has room (64 compute units idle in the last round,
// or a place each where two work-groups share one); 256 x 256 tiles never share, their column sums are a launch of their own.
inline bool dw_takes_colsum(int64_t d_in, int64_t d_out, int64_t k) {
    const int cfg = gemm_cfg(d_out, d_in, k);
    const int64_t tiles = gemm_tiles(cfg, d_out, d_in);
    if (cfg == GEMM_FEW || cfg == GEMM_SMALL || cfg == GEMM_FLAT) return tiles + colsum_blocks(d_out, 2) <= 512;  // (two on a compute unit)
    return (256 - tiles % 256) % 256 >= 64;
}

// Places for a work-group that the last round of a pass's paired launch leaves empty.
inline int64_t pair_idle(const PassPlan &p) {
    const int64_t slots = p.plain.cfg == GEMM_COMPACT ? 512 : 256;
    return (slots - (p.plain.tiles + p.sketch.shares()) % slots) % slots;
}

// Plan of a backward pass.  With a bias gradient that the launch of dW has no room for, short last slices
// that take the compute units its column sums need are given up (16384 x 1024 -> 4096, k = 1638: 208 sketch
// work-groups instead of 243).
inline PassPlan plan_backward(int64_t n, int64_t d_in, int64_t d_out, int64_t k, int kind, bool with_dbias, int64_t room = kMostSlices) {
    const PassPlan p = plan_pass(n, d_out, d_in, k, kind, room);
    if (!with_dbias || p.sketch.per_tail == 0 || p.sketch.slices < 2 || dw_takes_colsum(d_in, d_out, k) || pair_idle(p) >= 16) return p;
    PassPlan even = p;
    const int64_t units = (n + 63) / 64, len = (units + p.sketch.slices - 1) / p.sketch.slices;
    even.sketch.per_tail = 0, even.sketch.k_chunk = len * 64, even.sketch.slices = even.sketch.splits = (int)((units + len - 1) / len);
    return even.sketch.splits >= 2 && pair_idle(even) >= 16 ? even : p;
}

inline bool pass_pair_available(int64_t n, int64_t d_sk, int64_t d_other, int64_t k) {
    return k > kSmallK || small_pass_is_paired(n, d_sk, d_other, k);
}

// The two dense kinds may take different tiles and slices; a workspace serves either (and both plans of
// plan_backward: the one with a bias gradient has fewer slices).
inline size_t sketch_workspace_bf16(int64_t n, int64_t d, int64_t k, int64_t d_other = 0) {
    int64_t k_chunk;
    size_t most = 0;
    if (k <= kSmallK) {
        const int s = smallk_slices(n, d, k, &k_chunk);
        most = s > 1 ? (size_t)s * (size_t)k * (size_t)d * sizeof(float) : 0;
        if (d_other == 0 || !small_pass_is_paired(n, d, d_other, k)) return most;  // (no smaller than the streaming kernel's: without dX it runs all the same)
    }
    for (int kind = 0; kind < 2; ++kind) {
        const SketchPlan p = d_other > 0 ? plan_pass(n, d, d_other, k, kind).sketch : plan_sketch(n, d, k, kind, true);
        const size_t bytes = p.splits > 1 ? (size_t)p.splits * (size_t)k * (size_t)d * sizeof(float) : 0;
        if (bytes > most) most = bytes;
    }
    return most;
}
// The least that a pass runs in: two slices, or one where the partial sums are so many that the limited plan has one; of at most
// kSmallK columns what the streaming kernel takes (paired, such a pass makes do with fewer slices in that).
inline size_t least_sketch_workspace_bf16(int64_t n, int64_t d, int64_t k, int64_t d_other) {
    if (k <= kSmallK) return sketch_workspace_bf16(n, d, k);
    const size_t most = sketch_workspace_bf16(n, d, k, d_other);
    if (most == 0) return most;
    const bool sliced = plan_pass(n, d, d_other, k, 0, kLimited).sketch.splits > 1 || plan_pass(n, d, d_other, k, 1, kLimited).sketch.splits > 1;
    return sliced ? (size_t)2 * (size_t)k * (size_t)d * sizeof(float) : 0;
}

// ---- fp32 products, and bf16 products of widths the kernels above refuse (plain_kernels.hpp).
enum { PLAIN_BIG = 0, PLAIN_MID = 1, PLAIN_TINY = 2 };

// Tile shape of a plain product.  What counts is how evenly the tiles share the 256 compute units (one
// work-group each): the 128 x 128 tile where its last round costs no more than that of the 64 x 64 tile
// (it moves and splits half as many operand bytes per flop), the 64 x 64 tile otherwise, and below one
// 64 x 64 tile per compute unit the 32 x 32 tile, whose eight waves split the contraction.  fp32 operands are what
// splitting costs most: there a 128 x 128 tile takes 2.6 times as long as a 64 x 64 tile, not four times (dX 4096 x 3072 ->
// 768 with G beside it, k = 410: 328 -> 280 us; dW 768 -> 3072 38 -> 30).  `two_sums`: the 128 x 128 tile keeps two sums
// (plain_tile; dX and dW); with one, which is rounded twice as often, it stays where it was.  bf16 operands are not split:
// 64 x 64 tiles from 140 on (Y 700 x 300 -> 901, 165 tiles: 10.8 us on 32 x 32, 7.7 on 64 x 64; 500 x 1024 -> 1001, 128 tiles: 8.8 and
// 9.7), and of Y a 128 x 128 tile costs 2.8 of them (4096 x 1024 -> 1001: 23.9 and 18.4 us; dW 2048 x 1499, k = 1500: 58.9 and 60.0).
inline int plain_cfg(int elem_bytes, int64_t m, int64_t n, bool two_sums) {
    const int64_t big = tiles_of(m, n, 128, 128), mid = tiles_of(m, n, 64, 64);
    if (mid < (elem_bytes == 4 ? 256 : 140)) return PLAIN_TINY;
    const double times = elem_bytes == 4 ? (two_sums ? 2.6 : 4.0) : two_sums ? 4.0 : 2.8;
    return times * (double)((big + 255) / 256) <= (double)((mid + 255) / 256) ? PLAIN_BIG : PLAIN_MID;
}
// Tile of Y alone where X and W have rows on 16 bytes and Y has not: GEMM_COMPACT or GEMM_FLAT, which load straight into LDS and add in one order, in place
// of the 128 x 128 tile (`cfg`) and of 64 x 64 ones beyond a round of them; -1: that of `cfg`.  (3000 x 768 -> 1001 12.8 -> 10.0 us; 149 products of up to 4096
// tokens 0.878 of the time, three above 1.025, 1.06 at most.  Within a round their chain is longer: 1863 x 1976 -> 435, 210 tiles of 64 x 64 or 120 of 64 x 128, 12.8
// and 15.8.)
inline int any_width_tile(int cfg, int64_t m, int64_t n, int64_t kk) {
    if (cfg == PLAIN_TINY || (cfg == PLAIN_MID && (tiles_of(m, n, 64, 64) <= 256 || gemm_tiles(GEMM_FLAT, m, n) > 224))) return -1;
    if (cfg == PLAIN_MID) return GEMM_FLAT;  // (up to 224 of its tiles, half as many of 128 x 128 are never shorter)
    return gemm_us(GEMM_MID, m, n, kk) <= gemm_us(GEMM_FLAT, m, n, kk) ? GEMM_COMPACT : GEMM_FLAT;
}
inline int64_t plain_tiles(int cfg, int64_t m, int64_t n) {
    const int64_t e = cfg == PLAIN_BIG ? 128 : cfg == PLAIN_MID ? 64 : 32;
    return tiles_of(m, n, e, e);
}

// Whether an unsliced k x d sketch product beside plain tiles of `cfg` is on 32 x 32 tiles.  They generate every entry four times as often as
// 32 x 128 tiles: only where those are few.
inline bool plain_sketch_small(int cfg, int64_t k, int64_t d) {
    return cfg == PLAIN_TINY || (cfg == PLAIN_MID && tiles_of(k, d, 32, 128) < 64);
}

// Tile of dX beside G in an fp32 pass.  Beside 64 x 64 tiles few sketch tiles are 32 x 32, beside 128 x 128 tiles all are 32 x 128,
// which take 21 ns a token instead of 9 (+-1 entries 12.5 and 5.4): the larger tile only where that stays below what 64 x 64 tiles
// of dX take, half a round more than there are and 3.5 us and 18.5 ns a contraction element each (3308 x 609 -> 264, k = 331: backward
// 80 us with 128 x 128 tiles, 50 without; 3076 x 2776 -> 277, k = 615: 100 and 137).
inline int plain_backward_cfg_f32(int64_t n, int64_t d_in, int64_t d_out, int64_t k, int kind) {
    const int cfg = plain_cfg(4, n, d_in, true);
    if (cfg != PLAIN_BIG || plain_cfg(4, n, d_in, false) == PLAIN_BIG || tiles_of(k, d_out, 32, 128) >= 64) return cfg;
    const double rounds = (double)plain_tiles(PLAIN_MID, n, d_in) / 256 + 0.5;
    return (kind == 0 ? 21e-3 : 12.5e-3) * (double)n <= rounds * (3.5 + 18.5e-3 * (double)d_out) ? PLAIN_BIG : PLAIN_MID;
}

// How a launch loads its operands (rows of `a` and `b` elements): 4 = 16-byte loads (fp32, rows that start on 16
// bytes), 3 = rows that start anywhere, 0 = rows too long for 32-bit offsets inside a tile of 128 of them.  bf16 operands
// differ (rows_on_16): a row that starts anywhere costs a fifth dword, a funnel shift and its masks per eight
// elements (Y 3000 x 768 -> 1001 23 us with it, 17 without).
inline int load_mode(int elem_bytes, int64_t a, int64_t b) {
    const int64_t lim = (int64_t)1 << 22;
    if (a >= lim || b >= lim) return 0;
    return elem_bytes == 4 && a % 4 == 0 && b % 4 == 0 ? 4 : 3;
}
inline bool rows_on_16(int64_t row) { return row % 8 == 0; }  // bf16

// Token slices of a bf16 pass's sketch product: `slices` runs of `chunk` tokens, their fp32 sums `stride` elements apart in
// scratch.  One slice: no scratch.  `ld`: row length of the result and of the sums (0: as wide as the operand).  `cfg`: tile of
// the plain product of the pass (-1: none), which the sketch product's own tile depends on; the two take the same ones, `tile` included,
// launched one by one.
struct PlainSlices {
    int slices;
    int64_t chunk, stride, ld;
    int cfg;
    int tile = -1;  // (Y with rows that start anywhere: the tile of mfma_kernels.hpp in place of that of `cfg`, -1: none)
};

// Token slices of the sketch product of a bf16 pass (sketch of an n x d operand, beside a product n x d_other).  An entry is
// generated again for every column tile, and generating is most of what a Gaussian sketch tile does, so few wide tiles are
// wanted; slices make them many.  Modelled in us per pass, from what the tiles take alone: a 32 x 32 sketch tile 9 ns per token
// (+-1 entries 4.8), a 32 x 128 one 15 (9) and two on a compute unit 12 (6.5) each, a 64 x 64 tile of the other product 8 ns per
// contraction element, a 128 x 128 one 22 and a 32 x 32 one 6; a launch ends no sooner than its longest tile, nor than all its tiles on 256 compute
// units; slices add a launch of 4.5 us that reads their sums.  3000 x 768 -> 1001, Gaussian, k = 300: forward 43 us in one
// slice, 30 in two; backward 53, 43 in two.  4096 x 1024 -> 111, k = 205: backward 62, 20 in eleven.  Where the two come out
// alike (within 1 us) there are none.  At most `most`: what the caller's scratch holds.
inline PlainSlices plain_slices_beside(int cfg, int64_t n, int64_t d, int64_t k, int64_t d_other, int kind, int64_t most) {
    PlainSlices cut{1, n, 0, (d + 7) / 8 * 8, cfg};
    if (load_mode(2, d, d_other) == 0) return cut;
    const int64_t tiles = tiles_of(k, d, 32, 128);
    const double per_cu = 1.0 / 256, chain = (cfg == PLAIN_TINY ? 6e-3 : cfg == PLAIN_MID ? 8e-3 : 22e-3) * (double)d,
                 plain_work = chain * (double)plain_tiles(cfg, n, d_other) * per_cu;
    const double narrow = (kind == 0 ? 9e-3 : 4.8e-3) * (double)n, wide = (kind == 0 ? 15e-3 : 9e-3) * (double)n,
                 wide_work = (kind == 0 ? 12e-3 : 6.5e-3) * (double)n * (double)tiles;
    const bool small = plain_sketch_small(cfg, k, d);
    auto longest = [&](double sketch_chain, double sketch_work) {
        const double tile = sketch_chain > chain ? sketch_chain : chain, all = plain_work + sketch_work * per_cu;
        return tile > all ? tile : all;
    };
    double best = (small ? longest(narrow, narrow * (double)tiles_of(k, d, 32, 32)) : longest(wide, wide_work)) - 1.0;
    for (int64_t s = 2; s <= 16 && s <= most; ++s) {
        const int64_t chunk = ((n + s - 1) / s + 127) / 128 * 128, slices = (n + chunk - 1) / chunk;
        if (slices != s || chunk < 256) continue;
        const double t = longest(wide * (double)chunk / (double)n, wide_work) + 4.5 + 1e-6 * (double)(s * k * d);
        if (t < best) best = t, cut = PlainSlices{(int)s, chunk, k * cut.ld, cut.ld, cfg};
    }
    return cut;
}

// The tile of the plain product and the slices of a pass.  A launch of 128 x 128 tiles of Y and sketch tiles that goes a little over a
// round, by up to a quarter of the compute units, has most of them wait for the last few.  With 64 x 64 tiles, three rounds of
// them at most, the +-1 kind is 7 % faster there (81 random forward passes; 0.80 to 1.05 of the time; 3000 x 768 -> 1001, k = 300, 312
// work-groups: 22.4 and 20.7 us), the Gaussian kind, whose sketch tiles are longest by far, is not; nor are passes whose
// sketch product would lose more than half of its slices beside them (9 passes 1.01 to 1.49: 3495 x 400 -> 799, k = 174, four slices and
// one: 17.9 and 26.7 us).
inline PlainSlices plain_slices_on(int64_t n, int64_t d, int64_t k, int64_t d_other, int kind, bool backward, int64_t most = 16) {
    const PlainSlices cut = plain_slices_beside(plain_cfg(2, n, d_other, backward), n, d, k, d_other, kind, most);
    if (backward || kind != RMM_SKETCH_RADEMACHER || cut.cfg != PLAIN_BIG) return cut;
    const int64_t plain = plain_tiles(PLAIN_BIG, n, d_other), all = plain + tiles_of(k, d, 32, 128) * cut.slices;
    const bool short_round = plain <= 256 && all > 256 && all % 256 >= 1 && all % 256 <= 64;
    if (!short_round || plain_tiles(PLAIN_MID, n, d_other) > 768) return cut;
    const PlainSlices mid = plain_slices_beside(PLAIN_MID, n, d, k, d_other, kind, most);
    return 2 * mid.slices >= cut.slices ? mid : cut;
}

// The tile of Y beside a sketch product, rows of X and W on 16 bytes (as any_width_tile, which has Y alone).  In place of 128 x 128 tiles GEMM_COMPACT: 150 passes 0.945 of
// the time, 9 above 1.025 (with GEMM_FLAT where that alone is shorter 0.965 and 23).  In place of 64 x 64 ones GEMM_FLAT where with the sketch tiles each
// work-group has a compute unit to itself (72 passes: 0.87, none above 1.025), or where 64 x 64 tiles and sketch tiles go over two on each and no sketch tile takes
// 1.5 times as long as Y (`tile_ns` a token, as below; 70 passes 0.865, three above 1.025).  Elsewhere both have their places at once and last as long
// as the sketch tiles: 157 passes 0.997, 54 of them above 1.025, 1.15 at most (3688 x 2576 -> 277, k = 184, Rademacher, 28.4 -> 32.8 us).  500 fresh
// passes that one of these tiles is meant for: 0.938, 19 above 1.025, six of them above 1.1, 1.14 at most (1119 x 3168 -> 1857, k = 111, Rademacher, 35.1 ->
// 40.0: 128 x 128 tiles and sketch tiles one to nearly every compute unit, where GEMM_COMPACT has none beside it to fill its waits).
// Y with its sketch, 3000 x 768 -> 1001, k = 300: 25.3 -> 22.2 us; 1340 x 1080 -> 1217, k = 134, Rademacher, 16.1 -> 12.0.
inline int any_width_tile_beside(const PlainSlices &cut, int64_t n, int64_t d, int64_t k, int64_t d_other, int kind) {
    const int tile = any_width_tile(cut.cfg, n, d_other, d);
    if (tile < 0 || cut.cfg == PLAIN_BIG) return tile < 0 ? -1 : GEMM_COMPACT;
    const bool small = cut.slices <= 1 && plain_sketch_small(cut.cfg, k, d);
    const int64_t sketch = tiles_of(k, d, 32, small ? 32 : 128) * cut.slices;
    if (gemm_tiles(GEMM_FLAT, n, d_other) + sketch <= 256) return GEMM_FLAT;
    const double tile_ns = small ? (kind == 0 ? 9e-3 : 4.8e-3) : kind == 0 ? 15e-3 : 9e-3;
    const bool longest = tile_ns * (double)cut.chunk >= 1.5 * gemm_us(GEMM_FLAT, n, d_other, d);
    return plain_tiles(PLAIN_MID, n, d_other) + sketch > 512 && !longest ? GEMM_FLAT : -1;
}
inline PlainSlices plain_slices(int64_t n, int64_t d, int64_t k, int64_t d_other, int kind, bool backward, int64_t most = 16) {
    PlainSlices cut = plain_slices_on(n, d, k, d_other, kind, backward, most);
    if (!backward) cut.tile = any_width_tile_beside(cut, n, d, k, d_other, kind);
    return cut;
}

}  // namespace rmm
