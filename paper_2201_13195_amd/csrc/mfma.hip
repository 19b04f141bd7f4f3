// bf16 MFMA path of the RMM layer: which kernel of mfma_kernels.hpp serves which product at
// which shape, and the launches.
#include "../../include/rmm.h"
#include "mfma_pair.hpp"
#include "sors_kernels.hpp"

namespace rmm {

namespace {

int64_t tiles_of(int64_t m, int64_t n, int64_t bm, int64_t bn) { return ((m + bm - 1) / bm) * ((n + bn - 1) / bn); }

template <typename S>
int64_t tiles_in(int64_t m, int64_t n) { return tiles_of(m, n, S::BM, S::BN); }

// Time of a product on a menu of tiles, to choose between them (us, fitted to products from 256 x 384 to 16384 x 4096
// outputs and contractions from 51 to 4096): a launch, then rounds of 256 work-groups, each `fix` for the first loads and
// the writing of the tile and `step` for every 64 contraction elements.  Of the small tiles two share a compute unit: a
// full round of 512 takes 1.9 times the time of one of up to 256, one of 257 to 511 from 1.4 times on (`filled`, where other
// work-groups of the launch take the second places: 1.9 times too).
struct TileTime {
    int64_t bm, bn;
    double fix, step;
    bool shared;
};
double tile_us(const TileTime &t, int64_t m, int64_t n, int64_t kk, bool filled) {
    const int64_t tiles = tiles_of(m, n, t.bm, t.bn), rest = tiles % 512;
    const double rounds = !t.shared ? (double)((tiles + 255) / 256)
                                    : 1.9 * (double)(tiles / 512) + (rest == 0 ? 0.0 : rest <= 256 ? 1.0 : filled ? 1.9 : 1.4 + 0.5 * (double)(rest - 256) / 256.0);
    return 2.5 + rounds * (t.fix + (double)((kk + 63) / 64) * t.step);
}

// Tile of a plain product with an m x n output and contraction kk.  32 x 32 tiles whose contraction is shared by eight
// waves (few_tile) only while there are at most 512 of them.  256 x 256 tiles from 160 of them on whatever the model
// says: they need half the bytes per flop of 128 x 128 tiles, which a full chip cannot bring into its LDS at MFMA rate.
int gemm_cfg(int64_t m, int64_t n, int64_t kk, bool filled = false) {
    if (tiles_in<ShapeLarge>(m, n) >= 160) return GEMM_LARGE;
    static const struct {
        int cfg;
        TileTime t;
    } menu[] = {{GEMM_WIDE, {ShapeWide::BM, ShapeWide::BN, 3.0, 0.90, false}},
                {GEMM_SPLIT, {ShapeSplit::BM, ShapeSplit::BN, 2.4, 0.47, false}},
                {GEMM_MID, {ShapeMid::BM, ShapeMid::BN, 2.0, 0.50, false}},
                {GEMM_FLAT, {ShapeFlat::BM, ShapeFlat::BN, 1.0, 0.42, true}},
                {GEMM_SMALL, {ShapeSmall::BM, ShapeSmall::BN, 1.0, 0.27, true}}};
    int best = GEMM_FEW;
    double best_us = -1.0;
    const int64_t few = tiles_of(m, n, FewTile::E, FewTile::E);
    if (few <= 512)  // (two on a compute unit: where a wave's share is one step the second costs 0.6 of the first)
        best_us = 2.5 + (few <= 256 ? 1.0 : kk <= kFewSingle ? 1.6 : 2.0) * (1.0 + 0.85 * (double)kk / (double)kFewSingle);
    for (const auto &e : menu) {
        const double us = tile_us(e.t, m, n, kk, filled);
        if (best_us < 0.0 || us < best_us) best = e.cfg, best_us = us;
    }
    return best;
}

int64_t gemm_tiles(int cfg, int64_t m, int64_t n) {
    switch (cfg) {
        case GEMM_LARGE: return tiles_in<ShapeLarge>(m, n);
        case GEMM_WIDE: return tiles_in<ShapeWide>(m, n);
        case GEMM_SPLIT: return tiles_in<ShapeSplit>(m, n);
        case GEMM_COMPACT:
        case GEMM_MID: return tiles_in<ShapeMid>(m, n);
        case GEMM_FLAT: return tiles_in<ShapeFlat>(m, n);
        case GEMM_SMALL: return tiles_in<ShapeSmall>(m, n);
        default: return tiles_of(m, n, FewTile::E, FewTile::E);
    }
}

template <typename S, int AMODE, int BMODE, int OUT>
hipError_t launch(const GemmArgs &g, hipStream_t stream) {
    gemm_mfma_kernel<S, AMODE, BMODE, OUT><<<(unsigned)tiles_in<S>(g.M, g.N), S::THREADS, 0, stream>>>(g);
    return hipGetLastError();
}

template <int AMODE, int BMODE>
hipError_t launch_few(const GemmArgs &g, hipStream_t stream) {
    const unsigned grid = (unsigned)tiles_of(g.M, g.N, FewTile::E, FewTile::E);
    if (g.K <= kFewSingle)
        few_tile_kernel<AMODE, BMODE, true><<<grid, kFewThreads, 0, stream>>>(g);
    else
        few_tile_kernel<AMODE, BMODE, false><<<grid, kFewThreads, 0, stream>>>(g);
    return hipGetLastError();
}

template <int AMODE, int BMODE>
hipError_t launch_gemm(int cfg, const GemmArgs &g, hipStream_t stream) {
    switch (cfg) {
        case GEMM_LARGE: return launch<ShapeLarge, AMODE, BMODE, OUT_BF16>(g, stream);
        case GEMM_WIDE: return launch<ShapeWide, AMODE, BMODE, OUT_BF16>(g, stream);
        case GEMM_SPLIT: return launch<ShapeSplit, AMODE, BMODE, OUT_BF16>(g, stream);
        case GEMM_MID: return launch<ShapeMid, AMODE, BMODE, OUT_BF16>(g, stream);
        case GEMM_FLAT: return launch<ShapeFlat, AMODE, BMODE, OUT_BF16>(g, stream);
        case GEMM_SMALL: return launch<ShapeSmall, AMODE, BMODE, OUT_BF16>(g, stream);
        default: return launch_few<AMODE, BMODE>(g, stream);
    }
}

GemmArgs args_nt(const bf16_t *X, const bf16_t *W, const bf16_t *bias, bf16_t *Y, int64_t n, int64_t d_in, int64_t d_out) {
    GemmArgs g{};
    g.A = X, g.lda = d_in, g.B = W, g.ldb = d_in, g.C = Y, g.ldc = d_out, g.bias = bias;
    g.M = n, g.N = d_out, g.K = d_in, g.alpha = 1.0f;
    return g;
}

GemmArgs args_nn(const bf16_t *dY, const bf16_t *W, bf16_t *dX, int64_t n, int64_t d_in, int64_t d_out) {
    GemmArgs g{};
    g.A = dY, g.lda = d_out, g.B = W, g.ldb = d_in, g.C = dX, g.ldc = d_in, g.bias = nullptr;
    g.M = n, g.N = d_in, g.K = d_out, g.alpha = 1.0f;
    return g;
}

// Which kernel serves a sketch product with k > 64 and how its token dimension is cut.  The work-group
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
void slice_sketch(SketchPlan &p, int64_t n, int target_wgs, double overhead, int64_t most) {
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
        const int64_t tail_len = (int64_t)ceil(((double)units + overhead) * (double)m / (double)(s * m + 1));
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
const SketchMenu &sketch_menu(int cfg) {
    static const SketchMenu menu[kSketchTiles] = {{128, 256, {1.18, 0.91}}, {128, 512, {1.92, 1.63}}, {64, 512, {1.20, 1.04}},
                                                  {64, 384, {0.93, 0.86}},  {128, 384, {1.54, 1.30}}, {64, 256, {0.85, 0.61}}};
    return menu[cfg];  // (in the order of SK_NARROW ..)
}

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
// `limited`: the caller may be rmm_sketch_static.
SketchPlan plan_sketch(int64_t n, int64_t d, int64_t k, int kind, bool limited) {
    // rmm_sketch_static serves the shapes whose partial results fit RMM_STATIC_SCRATCH_BYTES with the plainest
    // tiling (rows by k, columns by d); those keep fitting, whichever tile they run with.
    int64_t most = 64;
    const double partial_bytes = (double)k * (double)d * 4.0;
    if (limited) {
        const int64_t tiles = d >= 1024 ? tiles_of(k, d, k <= 512 ? 64 : 128, 512) : d % 384 == 0 ? tiles_of(k, d, k <= 512 ? 64 : 128, 384) : tiles_of(k, d, 128, 256);
        const int64_t blocks = (n + 127) / 128, s = tiles >= 256 ? 1 : blocks < 256 / tiles ? blocks : 256 / tiles;
        const int64_t chunk = (blocks + s - 1) / s, slices = (blocks + chunk - 1) / chunk, fit = (int64_t)((double)RMM_STATIC_SCRATCH_BYTES / partial_bytes);
        if (slices == 1 || slices <= fit) most = fit < 1 ? 1 : fit < 64 ? fit : 64;
    }
    SketchPlan best{};
    double best_us = -1.0;
    static const int order[kSketchTiles] = {SK_WIDE64, SK_WIDE, SK_MID64, SK_MID, SK_NARROW64, SK_NARROW};
    for (int cfg : order) {
        const SketchMenu &e = sketch_menu(cfg);
        SketchPlan p;
        p.cfg = cfg, p.tiles = tiles_of(k, d, e.bm, e.bn);
        const double step_us = e.step_us[kind != 0];
        slice_sketch(p, n, 256, 4.0 / step_us, most);
        const double us = (double)((p.shares() + 255) / 256) * (double)(p.k_chunk / 64) * step_us + 2.0 * p.per_tail +
                          (p.splits > 1 ? (double)p.splits * (double)k * (double)d * 0.82e-6 : 0.0);
        if (best_us < 0.0 || us < 0.98 * best_us) best = p, best_us = us;  // (ties: the wider tile)
    }
    return best;
}

GemmArgs args_sketch(const bf16_t *A, int64_t n, int64_t d, int64_t k, SketchState st, const SketchPlan &p, bf16_t *out,
                     void *ws) {
    GemmArgs g{};
    g.A = nullptr, g.lda = 0, g.B = A, g.ldb = d, g.bias = nullptr;
    g.M = k, g.N = d, g.K = n, g.st = st, g.ldc = d, g.k_chunk = p.k_chunk, g.slices = p.slices, g.per_tail = p.per_tail;
    if (p.splits == 1) {
        g.C = out, g.alpha = 1.0f / sqrtf((float)k), g.direct = 1;
    } else {
        g.C = ws, g.alpha = 1.0f, g.split_stride = k * d;
    }
    return g;
}

template <typename S>
hipError_t launch_sketch_tile(int kind, const GemmArgs &g, const SketchPlan &p, hipStream_t stream) {
    if (kind == 0)
        sketch_kernel<S, 0><<<(unsigned)p.shares(), S::THREADS, 0, stream>>>(g, (int)p.tiles);
    else
        sketch_kernel<S, 1><<<(unsigned)p.shares(), S::THREADS, 0, stream>>>(g, (int)p.tiles);
    return hipGetLastError();
}

hipError_t launch_sketch_plan(const SketchPlan &p, int kind, const GemmArgs &g, hipStream_t stream) {
    switch (p.cfg) {
        case SK_WIDE: return launch_sketch_tile<ShapeSkWide>(kind, g, p, stream);
        case SK_WIDE64: return launch_sketch_tile<ShapeSkWide64>(kind, g, p, stream);
        case SK_MID64: return launch_sketch_tile<ShapeSkMid64>(kind, g, p, stream);
        case SK_MID: return launch_sketch_tile<ShapeSkMid>(kind, g, p, stream);
        case SK_NARROW64: return launch_sketch_tile<ShapeSkNarrow64>(kind, g, p, stream);
        default: return launch_sketch_tile<ShapeSkNarrow>(kind, g, p, stream);
    }
}

hipError_t launch_reduce(const void *ws, bf16_t *out, int64_t k, int64_t d, int splits, hipStream_t stream) {
    const int64_t elems = k * d;  // d % 8 == 0, so elems % 4 == 0
    reduce_partials_kernel<<<(unsigned)((elems / 4 + 255) / 256), 256, 0, stream>>>((const float *)ws, out, elems, splits,
                                                                                     elems, 1.0f / sqrtf((float)k));
    return hipGetLastError();
}

// The streaming kernel of small sketch sizes: token slices so that about one work-group per
// compute unit exists; 2 register sets of loads in flight.  Work-groups take 256 columns, or 128
// where that would leave slices of at most 2048 tokens (k <= 32) / 512 tokens (k <= 64): half as many,
// twice as long slices then halve the partial sums and the final cross-wave sum of a work-group
// (measured: 26.6 against 27.6 us at 16384 x 4096, k = 32; 11.7 against 15.3 us at 16384 x 1024),
// while on long slices the wider work-group is ahead (82.8 against 84.6 us at 65536 x 4096).
constexpr int64_t kSmallK = 64;
int smallk_slices_for(int64_t n, int64_t d, int64_t bn, int64_t *k_chunk) {
    const int64_t col_tiles = (d + bn - 1) / bn, blocks = (n + 127) / 128;
    int64_t s = 256 / col_tiles;
    if (s > blocks) s = blocks;
    if (s < 1) s = 1;
    *k_chunk = (blocks + s - 1) / s * 128;
    return (int)((n + *k_chunk - 1) / *k_chunk);
}
int64_t smallk_bn(int64_t n, int64_t d, int64_t k) {
    int64_t k_chunk;
    (void)smallk_slices_for(n, d, 256, &k_chunk);
    return k_chunk <= (k <= 32 ? 2048 : 512) ? 128 : 256;
}
int smallk_slices(int64_t n, int64_t d, int64_t k, int64_t *k_chunk) {
    return smallk_slices_for(n, d, smallk_bn(n, d, k), k_chunk);
}

template <int TM, int BN, int KIND>
hipError_t launch_smallk(const SmallkArgs &g, int slices, hipStream_t stream) {
    const dim3 grid((unsigned)((g.d + BN - 1) / BN), (unsigned)slices);
    if (slices == 1)
        sketch_smallk_kernel<TM, BN, KIND, 2, OUT_BF16><<<grid, 256, 0, stream>>>(g);
    else
        sketch_smallk_kernel<TM, BN, KIND, 2, OUT_F32_PARTIAL><<<grid, 256, 0, stream>>>(g);
    return hipGetLastError();
}

// Brackets a kernel with the caller's events (either may be null: nothing is recorded).
struct EventPair {
    hipEvent_t begin, end;
    hipStream_t stream;
    EventPair(hipEvent_t b, hipEvent_t e, hipStream_t s) : begin(b), end(e), stream(s) {
        if (begin != nullptr && end != nullptr) (void)hipEventRecord(begin, stream);
    }
    void done() {
        if (begin != nullptr && end != nullptr) (void)hipEventRecord(end, stream);
        begin = end = nullptr;
    }
    ~EventPair() { done(); }
};

// ---- Paired launches: which tiles and slices a pass takes.

// Time until `second` jobs of t2 us each are done that follow `first` jobs of t1 us on `slots` equal slots.
double makespan(int64_t first, double t1, int64_t second, double t2, int64_t slots) {
    const int64_t late = first % slots, early = slots - late;  // slots that become free a round later / at once
    const double base = (double)(first / slots) * t1;
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

// us of a paired launch and the sum of its slices: work-groups of either kind take a time of their own (first loads and
// writing, and every step of 64 contraction elements) and are dealt to 256 slots in grid order, or to 512 where two share
// a compute unit.  The times are fitted to 4300 launches of 60 passes (256 to 16384 tokens, widths 256 to 4096,
// k = 73 to 6911; all sketch tiles, 64 to 512 work-groups): 7 % rms off.  Over those passes the plan it leads to is 3.3 % slower than the
// best one on average and 30 % at most; plans made for the sketch product alone were 12 and 50 %.
double pair_us(const PairPlain &plain, int64_t kk, const SketchPlan &p, int kind, double partial_mb) {
    struct Times {
        double fix, step;
    };
    static const Times large{6.3, 1.405}, split{4.0, 0.478}, mid{3.4, 0.487}, compact{5.4, 0.733};
    struct SketchTimes {
        double fix, step[2];  // Gaussian, Rademacher
    };
    static const SketchTimes sk_compact{5.5, {1.009, 0.935}};
    static const SketchTimes sk[] = {{5.3, {1.288, 0.957}}, {7.2, {1.651, 1.476}}, {5.1, {1.078, 1.080}},   // (in the order of SK_NARROW ..)
                                     {5.0, {0.929, 0.910}}, {6.3, {1.490, 1.192}}, {4.05, {0.780, 0.722}}};
    const bool two = plain.cfg == GEMM_COMPACT;
    const Times &a = plain.cfg == GEMM_LARGE ? large : plain.cfg == GEMM_SPLIT ? split : two ? compact : mid;
    const SketchTimes &b = two ? sk_compact : sk[p.cfg];
    const double ta = a.fix + a.step * (double)((kk + 63) / 64), tb = b.fix + b.step[kind != 0] * (double)(p.k_chunk / 64);
    const int64_t slots = two ? 512 : 256;
    double t = sketch_goes_first(plain.tiles, p.slices) ? makespan(p.shares(), tb, plain.tiles, ta, slots)
                                                        : makespan(plain.tiles, ta, p.shares(), tb, slots);
    // Beside 256 x 256 tiles, several rounds of them, power limits the chip's clock and a sketch work-group as long as the launch takes a
    // tenth more (16384 x 1024 -> 4096, k = 1638, Rademacher: 78 work-groups of 169 us by the times above 202 us with the sum of the
    // slices, 91 of 115 185).
    if (plain.cfg == GEMM_LARGE && plain.tiles > 256 && t < 1.1 * tb) t = 1.1 * tb;
    return t + (p.splits > 1 ? 2.6 + 0.213 * (double)p.splits * partial_mb : 0.0);
}

struct PassPlan {
    PairPlain plain;
    SketchPlan sketch;
};

// The plain product of a pass (contraction kk, n x m outputs) beside a sketch product on one work-group per compute unit:
// 256 x 256 tiles where it fills the chip with them, else 128 x 128; with two wave groups where the contraction is long (4096 x
// 3072 -> 768 alone: 25.0 us, without 25.5; 768 -> 768: 10.3, without 9.7).
PairPlain pair_plain(int64_t n, int64_t m, int64_t kk) {
    const int cfg = tiles_in<ShapeLarge>(n, m) >= 160 ? GEMM_LARGE : kk >= 1536 ? GEMM_SPLIT : GEMM_MID;
    return PairPlain{cfg, (int)gemm_tiles(cfg, n, m)};
}

// Plan of a pass: sketch of the n x d_sk operand, plain product n x d_other over d_sk.  Every sketch tile with slices for 64
// to 320 work-groups, and 64 x 256 tiles with ShapeCompact where all work-groups are resident at once.  (4096 x 768 ->
// 768, k = 410, with the sum of its slices: 26.9 -> 21.3 us; 4096 x 3072 -> 768, k = 2048, Rademacher 82 -> 69; 3001 x 1304 ->
// 520, k = 600: 32 -> 24.)  At most a quarter more slices than alone: no pass needs much more workspace than its sketch
// product.  Less than 0.8 us, which is what the model is off by at the smallest sizes, is not worth another order of additions
// than that of the product alone.
PassPlan make_pass_plan(int64_t n, int64_t d_sk, int64_t d_other, int64_t k, int kind) {
    const SketchPlan alone = plan_sketch(n, d_sk, k, kind, true);
    const double partial_mb = (double)k * (double)d_sk * 4e-6;
    const PairPlain usual = pair_plain(n, d_other, d_sk);
    const PairPlain compact{GEMM_COMPACT, (int)gemm_tiles(GEMM_COMPACT, n, d_other)};
    PassPlan best{usual, alone};
    double best_us = pair_us(usual, d_sk, alone, kind, partial_mb) - 0.8;
    for (int cfg = 0; cfg < kSketchTiles; ++cfg) {
        int slices = -1, per_tail = -1;
        for (int target : {64, 96, 128, 192, 256, 320}) {
            SketchPlan p;
            p.cfg = cfg, p.tiles = tiles_of(k, d_sk, sketch_menu(cfg).bm, sketch_menu(cfg).bn);
            slice_sketch(p, n, target, 4.0 / sketch_menu(cfg).step_us[kind != 0], 64);
            if (p.slices == slices && p.per_tail == per_tail) continue;
            slices = p.slices, per_tail = p.per_tail;
            if (p.splits > 1 && (alone.splits == 1 || 4 * (p.splits - 1) > 5 * alone.splits)) continue;
            double us = pair_us(usual, d_sk, p, kind, partial_mb);
            if (us < best_us) best = PassPlan{usual, p}, best_us = us;
            if (cfg != SK_NARROW64 || usual.cfg == GEMM_LARGE || compact.tiles + p.shares() > 512) continue;
            us = pair_us(compact, d_sk, p, kind, partial_mb);
            if (us < best_us) best = PassPlan{compact, p}, best_us = us;
        }
    }
    return best;
}

// The same, remembered: a pass asks for its plan three times (workspace of either kind, launch), and it depends on the
// sizes alone.
PassPlan plan_pass(int64_t n, int64_t d_sk, int64_t d_other, int64_t k, int kind) {
    struct Entry {
        int64_t n, d_sk, d_other, k;
        int kind;
        PassPlan plan;
    };
    constexpr size_t ENTRIES = 64;
    static thread_local Entry memo[ENTRIES];  // (n = 0: empty)
    kind = kind != 0;
    const uint64_t h = ((uint64_t)n * 0x9E3779B97F4A7C15u ^ (uint64_t)d_sk * 0xC2B2AE3D27D4EB4Fu ^ (uint64_t)d_other * 0x165667B19E3779F9u ^
                        (uint64_t)k * 0x27D4EB2F165667C5u) + (uint64_t)kind;
    Entry &e = memo[(h ^ h >> 32) % ENTRIES];
    if (e.n != n || e.d_sk != d_sk || e.d_other != d_other || e.k != k || e.kind != kind)
        e = Entry{n, d_sk, d_other, k, kind, make_pass_plan(n, d_sk, d_other, k, kind)};
    return e.plan;
}

// Whether the launch of dW has room for the column sums of the bias gradient beside it.
bool dw_takes_colsum(int64_t d_in, int64_t d_out, int64_t k) {
    const int cfg = gemm_cfg(d_out, d_in, k);
    const int64_t tiles = gemm_tiles(cfg, d_out, d_in);
    if (cfg == GEMM_FEW || cfg == GEMM_SMALL || cfg == GEMM_FLAT) return tiles + colsum_blocks(d_out, 2) <= 512;  // (two on a compute unit)
    return (256 - tiles % 256) % 256 >= 64;
}

// Places for a work-group that the last round of a pass's paired launch leaves empty.
int64_t pair_idle(const PassPlan &p) {
    const int64_t slots = p.plain.cfg == GEMM_COMPACT ? 512 : 256;
    return (slots - (p.plain.tiles + p.sketch.shares()) % slots) % slots;
}

// Plan of a backward pass.  With a bias gradient that the launch of dW has no room for, short last slices
// that take the compute units its column sums need are given up (16384 x 1024 -> 4096, k = 1638: 208 sketch
// work-groups instead of 243).
PassPlan plan_backward(int64_t n, int64_t d_in, int64_t d_out, int64_t k, int kind, bool with_dbias) {
    const PassPlan p = plan_pass(n, d_out, d_in, k, kind);
    if (!with_dbias || p.sketch.per_tail == 0 || p.sketch.slices < 2 || dw_takes_colsum(d_in, d_out, k) || pair_idle(p) >= 16) return p;
    PassPlan even = p;
    const int64_t units = (n + 63) / 64, len = (units + p.sketch.slices - 1) / p.sketch.slices;
    even.sketch.per_tail = 0, even.sketch.k_chunk = len * 64, even.sketch.slices = even.sketch.splits = (int)((units + len - 1) / len);
    return even.sketch.splits >= 2 && pair_idle(even) >= 16 ? even : p;
}

}  // namespace

bool mfma_shape_ok(int64_t n, int64_t d_in, int64_t d_out, int64_t k) {
    // 16-byte chunks need widths that are multiples of 8; a buffer descriptor spans up to 256 rows
    // of an operand with 32-bit byte offsets, so a row has to stay below 2^22 elements.  The token
    // count and the sketch size are not limited here (operands of 2 GiB and more are fine).
    (void)n, (void)k;
    const int64_t lim = (int64_t)1 << 22;
    return d_in % 8 == 0 && d_out % 8 == 0 && d_in < lim && d_out < lim;
}

// `pair_k`, if not 0: with the tiles the product has in its pass's paired launch with a sketch of pair_k columns, so that a
// pass whose products are launched one by one (to be timed) gives the same bits.  (ShapeCompact adds in ShapeMid's order.)
template <int BMODE>
static hipError_t launch_plain_of_pass(const GemmArgs &g, int64_t pair_k, int kind, hipStream_t stream) {
    if (pair_k == 0) return launch_gemm<A_KCONTIG, BMODE>(gemm_cfg(g.M, g.N, g.K), g, stream);
    const int cfg = (kind == RMM_SKETCH_SORS ? pair_plain(g.M, g.N, g.K) : plan_pass(g.M, g.K, g.N, pair_k, kind).plain).cfg;
    return launch_gemm<A_KCONTIG, BMODE>(cfg == GEMM_COMPACT ? GEMM_MID : cfg, g, stream);
}

hipError_t launch_linear_nt_bf16(const bf16_t *X, const bf16_t *W, const bf16_t *bias, bf16_t *Y, int64_t n,
                                 int64_t d_in, int64_t d_out, int64_t pair_k, int kind, hipStream_t stream) {
    return launch_plain_of_pass<B_KCONTIG>(args_nt(X, W, bias, Y, n, d_in, d_out), pair_k, kind, stream);
}

hipError_t launch_linear_nn_bf16(const bf16_t *dY, const bf16_t *W, bf16_t *dX, int64_t n, int64_t d_in,
                                 int64_t d_out, int64_t pair_k, int kind, hipStream_t stream) {
    return launch_plain_of_pass<B_NCONTIG>(args_nn(dY, W, dX, n, d_in, d_out), pair_k, kind, stream);
}

hipError_t launch_dw_bf16(const bf16_t *G, const bf16_t *X_proj, bf16_t *dW, int64_t k, int64_t d_in, int64_t d_out,
                          hipStream_t stream, bool accumulate) {
    GemmArgs g{};
    g.accumulate = accumulate ? 1 : 0;
    g.A = G, g.lda = d_out, g.B = X_proj, g.ldb = d_in, g.C = dW, g.ldc = d_in, g.bias = nullptr;
    g.M = d_out, g.N = d_in, g.K = k, g.alpha = 1.0f;
    return launch_gemm<A_MCONTIG, B_NCONTIG>(gemm_cfg(g.M, g.N, g.K), g, stream);
}

template <typename S>
static hipError_t launch_dw_colsum(const GemmArgs &g, const ColsumArgs &c, hipStream_t stream) {
    const int blocks_a = (int)tiles_in<S>(g.M, g.N);
    dw_colsum_kernel<S><<<(unsigned)(blocks_a + colsum_blocks(c.d, 2)), S::THREADS, 0, stream>>>(g, c, blocks_a);
    return hipGetLastError();
}

static hipError_t launch_few_dw_colsum(const GemmArgs &g, const ColsumArgs &c, hipStream_t stream) {
    const int blocks_a = (int)tiles_of(g.M, g.N, FewTile::E, FewTile::E);
    const unsigned grid = (unsigned)(blocks_a + colsum_blocks(c.d, 2));
    if (g.K <= kFewSingle)
        few_dw_colsum_kernel<true><<<grid, kFewThreads, 0, stream>>>(g, c, blocks_a);
    else
        few_dw_colsum_kernel<false><<<grid, kFewThreads, 0, stream>>>(g, c, blocks_a);
    return hipGetLastError();
}

hipError_t launch_dw_colsum_bf16(const bf16_t *G, const bf16_t *X_proj, bf16_t *dW, int64_t k, int64_t d_in, int64_t d_out,
                                 const bf16_t *dY, bf16_t *dbias, int64_t n, hipStream_t stream, bool accumulate) {
    GemmArgs g{};
    g.accumulate = accumulate ? 1 : 0;
    g.A = G, g.lda = d_out, g.B = X_proj, g.ldb = d_in, g.C = dW, g.ldc = d_in, g.bias = nullptr;
    g.M = d_out, g.N = d_in, g.K = k, g.alpha = 1.0f;
    const ColsumArgs c{dY, dbias, n, d_out, accumulate ? 1 : 0, colsum_lpr(d_out, 2)};
    switch (gemm_cfg(g.M, g.N, g.K)) {  // the tile dW runs with on its own
        case GEMM_LARGE: {  // 160 or more tiles of 256 x 256: dW fills the chip, the column sums follow as a launch of their own
            const hipError_t e = launch_dw_bf16(G, X_proj, dW, k, d_in, d_out, stream, accumulate);
            return e != hipSuccess ? e : launch_colsum<bf16_t>(dY, dbias, n, d_out, stream, accumulate);
        }
        case GEMM_WIDE: return launch_dw_colsum<ShapeWide>(g, c, stream);
        case GEMM_SPLIT: return launch_dw_colsum<ShapeSplit>(g, c, stream);
        case GEMM_MID: return launch_dw_colsum<ShapeMid>(g, c, stream);
        case GEMM_FLAT: return launch_dw_colsum<ShapeFlat>(g, c, stream);
        case GEMM_SMALL: return launch_dw_colsum<ShapeSmall>(g, c, stream);
        default: return launch_few_dw_colsum(g, c, stream);
    }
}

// |X^T dY|_F^2 per tile for the variance monitors: the dW-type product (both operands stored
// [token][feature]) with the squared-norm epilogue; the tiles of the other products, but for 32 x 32, beside the work-groups of
// the row norms (6670 tokens, 608 x 1704: 270 tiles of 64 x 64 63 us, 140 of 64 x 128 49).
static int xty_cfg(int64_t m, int64_t n, int64_t kk) {
    const int cfg = gemm_cfg(m, n, kk, true);
    return cfg == GEMM_FEW ? GEMM_SMALL : cfg;
}

int xty_sumsq_tiles(int64_t n, int64_t d_in, int64_t d_out) { return (int)gemm_tiles(xty_cfg(d_in, d_out, n), d_in, d_out); }

template <typename S>
static hipError_t launch_xty_norms(const GemmArgs &g, const RowNormArgs &r, hipStream_t stream) {
    const int tiles = (int)tiles_in<S>(g.M, g.N);
    xty_norms_kernel<S><<<(unsigned)(tiles + row_norm_blocks(r.n)), S::THREADS, 0, stream>>>(g, r, tiles);
    return hipGetLastError();
}

hipError_t launch_xty_norms_bf16(const bf16_t *X, const bf16_t *dY, double *part, double *rows, int64_t n, int64_t d_in,
                                 int64_t d_out, hipStream_t stream) {
    GemmArgs g{};
    g.A = X, g.lda = d_in, g.B = dY, g.ldb = d_out, g.C = part, g.ldc = d_out, g.bias = nullptr;
    g.M = d_in, g.N = d_out, g.K = n, g.alpha = 1.0f;
    const RowNormArgs r{X, dY, n, d_in, d_out, 1, rows};
    switch (xty_cfg(g.M, g.N, g.K)) {
        case GEMM_LARGE: return launch_xty_norms<ShapeLarge>(g, r, stream);
        case GEMM_WIDE: return launch_xty_norms<ShapeWide>(g, r, stream);
        case GEMM_SPLIT: return launch_xty_norms<ShapeSplit>(g, r, stream);
        case GEMM_MID: return launch_xty_norms<ShapeMid>(g, r, stream);
        case GEMM_FLAT: return launch_xty_norms<ShapeFlat>(g, r, stream);
        default: return launch_xty_norms<ShapeSmall>(g, r, stream);
    }
}

// The two dense kinds may take different tiles and slices; a workspace serves either (and both plans of
// plan_backward: the one with a bias gradient has fewer slices).
size_t sketch_workspace_bf16(int64_t n, int64_t d, int64_t k, int64_t d_other) {
    int64_t k_chunk;
    size_t most = 0;
    if (k <= kSmallK) {
        const int s = smallk_slices(n, d, k, &k_chunk);
        return s > 1 ? (size_t)s * (size_t)k * (size_t)d * sizeof(float) : 0;
    }
    for (int kind = 0; kind < 2; ++kind) {
        const SketchPlan p = d_other > 0 ? plan_pass(n, d, d_other, k, kind).sketch : plan_sketch(n, d, k, kind, true);
        const size_t bytes = p.splits > 1 ? (size_t)p.splits * (size_t)k * (size_t)d * sizeof(float) : 0;
        if (bytes > most) most = bytes;
    }
    return most;
}

hipError_t launch_sketch_bf16(const bf16_t *A, bf16_t *out, int64_t n, int64_t d, int64_t k, int kind, SketchState st,
                              void *ws, hipStream_t stream, hipEvent_t ev_begin, hipEvent_t ev_end, int64_t d_other,
                              bool with_dbias) {
    EventPair pev(ev_begin, ev_end, stream);
    if (k <= kSmallK) {  // bound by one pass over A: streaming kernel
        SmallkArgs a{};
        a.A = A, a.n = n, a.d = d, a.k = k, a.st = st;
        const int slices = smallk_slices(n, d, k, &a.k_chunk);
        a.C = slices == 1 ? (void *)out : ws, a.alpha = 1.0f / sqrtf((float)k);
        const bool narrow = smallk_bn(n, d, k) == 128;
        hipError_t e;
        if (k <= 32)
            e = narrow ? (kind == 0 ? launch_smallk<1, 128, 0>(a, slices, stream) : launch_smallk<1, 128, 1>(a, slices, stream))
                       : (kind == 0 ? launch_smallk<1, 256, 0>(a, slices, stream) : launch_smallk<1, 256, 1>(a, slices, stream));
        else
            e = narrow ? (kind == 0 ? launch_smallk<2, 128, 0>(a, slices, stream) : launch_smallk<2, 128, 1>(a, slices, stream))
                       : (kind == 0 ? launch_smallk<2, 256, 0>(a, slices, stream) : launch_smallk<2, 256, 1>(a, slices, stream));
        pev.done();
        if (e != hipSuccess || slices == 1) return e;
        return launch_reduce(ws, out, k, d, slices, stream);
    }
    const SketchPlan p = with_dbias    ? plan_backward(n, d_other, d, k, kind, true).sketch
                         : d_other > 0 ? plan_pass(n, d, d_other, k, kind).sketch
                                       : plan_sketch(n, d, k, kind, true);
    const GemmArgs g = args_sketch(A, n, d, k, st, p, out, ws);
    hipError_t e = launch_sketch_plan(p, kind, g, stream);
    pev.done();
    if (e != hipSuccess || p.splits == 1) return e;
    return launch_reduce(ws, out, k, d, p.splits, stream);
}

bool pass_pair_available(int64_t k) { return k > kSmallK; }

hipError_t launch_forward_pair_bf16(const bf16_t *X, const bf16_t *W, const bf16_t *bias, bf16_t *Y, bf16_t *X_proj,
                                    int64_t n, int64_t d_in, int64_t d_out, int64_t k, int kind, SketchState st, void *ws,
                                    hipStream_t stream, hipEvent_t ev_begin, hipEvent_t ev_end) {
    const GemmArgs ga = args_nt(X, W, bias, Y, n, d_in, d_out);
    const PassPlan pass = plan_pass(n, d_in, d_out, k, kind);
    const SketchPlan &p = pass.sketch;
    const GemmArgs gb = args_sketch(X, n, d_in, k, st, p, X_proj, ws);
    EventPair pev(ev_begin, ev_end, stream);
    const hipError_t e = launch_pair_nt(pass.plain, p.cfg, kind, ga, gb, (int)p.tiles, p.shares(), stream);
    pev.done();
    if (e != hipSuccess || p.splits == 1) return e;
    return launch_reduce(ws, X_proj, k, d_in, p.splits, stream);
}

// Where the bias gradient goes in a backward pass that has the paired launch: into the launch of
// dW when that leaves at least 64 compute units idle (dW is short and mostly latency; where it runs on
// few_tile, whose work-groups want a compute unit each, when the column blocks fit beside them);
// otherwise into the paired launch when its last round leaves at least 16 idle (the sketch work-groups
// of that round run for long, and dY is being read there anyway; plan_backward sees to it where it
// can); otherwise into the launch of dW.
bool backward_pair_takes_colsum(int64_t n, int64_t d_in, int64_t d_out, int64_t k, int kind) {
    if (!pass_pair_available(k)) return false;
    return !dw_takes_colsum(d_in, d_out, k) &&
           (gemm_cfg(d_out, d_in, k) == GEMM_FEW ||
            pair_idle(plan_backward(n, d_in, d_out, k, kind, true)) >= 16);
}

hipError_t launch_backward_pair_bf16(const bf16_t *dY, const bf16_t *W, bf16_t *dX, bf16_t *G, int64_t n, int64_t d_in,
                                     int64_t d_out, int64_t k, int kind, SketchState st, void *ws, hipStream_t stream,
                                     hipEvent_t ev_begin, hipEvent_t ev_end, bool with_dbias, bf16_t *dbias,
                                     bool accumulate_dbias) {
    const GemmArgs ga = args_nn(dY, W, dX, n, d_in, d_out);
    const PassPlan pass = plan_backward(n, d_in, d_out, k, kind, with_dbias);
    const SketchPlan &p = pass.sketch;
    const GemmArgs gb = args_sketch(dY, n, d_out, k, st, p, G, ws);
    const ColsumArgs gc{dY, dbias, n, d_out, accumulate_dbias ? 1 : 0, colsum_lpr(d_out, 2)};
    const ColsumArgs *gcp = dbias != nullptr ? &gc : nullptr;
    EventPair pev(ev_begin, ev_end, stream);
    const hipError_t e = launch_pair_nn(pass.plain, p.cfg, kind, ga, gb, (int)p.tiles, p.shares(), stream, gcp);
    pev.done();
    if (e != hipSuccess || p.splits == 1) return e;
    return launch_reduce(ws, G, k, d_out, p.splits, stream);
}

// ---- SORS kind: the plain product of a pass together with the strips of its sketch product.
// Worth it when the plain product leaves at least 32 compute units idle in its last round (the
// sketch work-groups need a compute unit to themselves); the strip kernel's chunked form must
// apply (at least 4096 tokens after padding, at most 2048 sketch columns).
static int sors_chunks(int64_t n) {
    int l = 0;
    while (((int64_t)1 << l) < n) ++l;
    return l >= 12 ? 1 << (l - 11) : 0;
}

// 0: separate launches; 1: strips behind the plain tiles (they fill the compute units its last
// round leaves idle, at least 32 of them); 2: strips in front (the plain product runs three or more
// rounds and the strips, few and long, occupy at most a quarter of the chip beside its first rounds).
static int sors_pair_order(int64_t blocks_a, int64_t strip_groups) {
    if ((256 - blocks_a % 256) % 256 >= 32) return 1;
    if (blocks_a >= 256 && strip_groups <= 64) return 2;
    return 0;
}

bool sors_pair_available(int64_t n, int64_t d_sk, int64_t d_other, int64_t k) {
    if (!sors_fast_ok(n, d_sk) || sors_chunks(n) == 0 || k > 2048) return false;
    const PairPlain plain = pair_plain(n, d_other, d_sk);
    // 128 x 128 tiles: one round of them, long enough for the strips to finish beside it
    if (plain.cfg != GEMM_LARGE && (plain.tiles < 65 || plain.tiles > 256 || d_sk < 768)) return false;
    return sors_pair_order(plain.tiles, (d_sk / 8 + 1) / 2) != 0;
}

static hipError_t launch_pass_sors(const GemmArgs &ga, bool row_indexed_b, const SorsArgs &gs, hipStream_t stream, hipEvent_t ev_begin,
                                   hipEvent_t ev_end) {
    const PairPlain plain = pair_plain(ga.M, ga.N, ga.K);
    EventPair pev(ev_begin, ev_end, stream);
    return launch_pair_sors(plain, row_indexed_b, ga, gs, sors_chunks(gs.n), sors_pair_order(plain.tiles, (gs.d / 8 + 1) / 2) == 2, stream);
}

hipError_t launch_forward_pair_sors_bf16(const bf16_t *X, const bf16_t *W, const bf16_t *bias, bf16_t *Y, bf16_t *X_proj,
                                         int64_t n, int64_t d_in, int64_t d_out, int64_t k, SketchState st,
                                         hipStream_t stream, hipEvent_t ev_begin, hipEvent_t ev_end) {
    const SorsArgs gs{X, X_proj, n, d_in, k, st, 1.0f / sqrtf((float)k), nullptr, 0};
    return launch_pass_sors(args_nt(X, W, bias, Y, n, d_in, d_out), false, gs, stream, ev_begin, ev_end);
}

hipError_t launch_backward_pair_sors_bf16(const bf16_t *dY, const bf16_t *W, bf16_t *dX, bf16_t *G, int64_t n,
                                          int64_t d_in, int64_t d_out, int64_t k, SketchState st, bf16_t *dbias,
                                          bool accumulate_dbias, hipStream_t stream, hipEvent_t ev_begin, hipEvent_t ev_end) {
    const SorsArgs gs{dY, G, n, d_out, k, st, 1.0f / sqrtf((float)k), dbias, accumulate_dbias ? 1 : 0};
    return launch_pass_sors(args_nn(dY, W, dX, n, d_in, d_out), true, gs, stream, ev_begin, ev_end);
}

}  // namespace rmm
