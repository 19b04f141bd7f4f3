// bf16 MFMA path of the RMM layer: the launches of the kernels of mfma_kernels.hpp (launch_plans.hpp: which one, and how it is cut).
#include "mfma_pair.hpp"
#include "sors_kernels.hpp"

namespace rmm {

namespace {

template <typename S>
int64_t tiles_in(int64_t m, int64_t n) { return tiles_of(m, n, S::BM, S::BN); }

// The plans count tiles of these edges.
template <typename S>
constexpr bool has_edges(int cfg) { return S::BM == kGemmTiles[cfg].bm && S::BN == kGemmTiles[cfg].bn; }
static_assert(has_edges<ShapeLarge>(GEMM_LARGE) && has_edges<ShapeWide>(GEMM_WIDE) && has_edges<ShapeSplit>(GEMM_SPLIT) && has_edges<ShapeMid>(GEMM_MID) &&
              has_edges<ShapeFlat>(GEMM_FLAT) && has_edges<ShapeSmall>(GEMM_SMALL) && has_edges<ShapeCompact>(GEMM_COMPACT), "tiles of the menu");
template <typename S>
constexpr bool has_sketch_edges(int cfg) { return S::BM == kSketchMenu[cfg].bm && S::BN == kSketchMenu[cfg].bn; }
static_assert(has_sketch_edges<ShapeSkNarrow>(SK_NARROW) && has_sketch_edges<ShapeSkWide>(SK_WIDE) && has_sketch_edges<ShapeSkWide64>(SK_WIDE64) &&
              has_sketch_edges<ShapeSkMid64>(SK_MID64) && has_sketch_edges<ShapeSkMid>(SK_MID) && has_sketch_edges<ShapeSkNarrow64>(SK_NARROW64), "sketch tiles");
static_assert(FewTile::E == kGemmTiles[GEMM_FEW].bm && FewTile::E == kGemmTiles[GEMM_FEW].bn && kFewSingle == 8 * FewTile::BK, "few_tile");

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

}  // namespace

// `pair_k`, if not 0: with the tiles the product has in its pass's paired launch with a sketch of pair_k columns, so that a
// pass whose products are launched one by one (to be timed) gives the same bits.  (ShapeCompact adds in ShapeMid's order.)
template <int BMODE>
static hipError_t launch_plain_of_pass(const GemmArgs &g, int64_t pair_k, int kind, int64_t room, hipStream_t stream) {
    if (pair_k == 0) return launch_gemm<A_KCONTIG, BMODE>(gemm_cfg(g.M, g.N, g.K), g, stream);
    const int cfg = (kind == RMM_SKETCH_SORS ? plan_sors(g.M, g.K, g.N, pair_k).plain : plan_pass(g.M, g.K, g.N, pair_k, kind, room).plain).cfg;
    return launch_gemm<A_KCONTIG, BMODE>(cfg == GEMM_COMPACT ? GEMM_MID : BMODE == B_NCONTIG ? dx_cfg(cfg, g.K) : cfg, g, stream);
}

hipError_t launch_linear_nt_bf16(const bf16_t *X, const bf16_t *W, const bf16_t *bias, bf16_t *Y, int64_t n,
                                 int64_t d_in, int64_t d_out, int64_t pair_k, int kind, int64_t room, hipStream_t stream) {
    return launch_plain_of_pass<B_KCONTIG>(args_nt(X, W, bias, Y, n, d_in, d_out), pair_k, kind, room, stream);
}

hipError_t launch_linear_nn_bf16(const bf16_t *dY, const bf16_t *W, bf16_t *dX, int64_t n, int64_t d_in,
                                 int64_t d_out, int64_t pair_k, int kind, int64_t room, hipStream_t stream) {
    return launch_plain_of_pass<B_NCONTIG>(args_nn(dY, W, dX, n, d_in, d_out), pair_k, kind, room, stream);
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

template <typename S>
static hipError_t launch_xty_norms(const GemmArgs &g, const RowNormArgs &r, hipStream_t stream) {
    const int tiles = (int)tiles_in<S>(g.M, g.N);
    xty_norms_kernel<S><<<(unsigned)(tiles + row_norm_blocks(r.n)), S::THREADS, 0, stream>>>(g, r, tiles);
    return hipGetLastError();
}

hipError_t launch_xty_norms_bf16(const bf16_t *X, const bf16_t *dY, double *part, double *rows, int64_t n, int64_t d_in,
                                 int64_t d_out, int64_t room, hipStream_t stream) {
    GemmArgs g{};
    g.A = X, g.lda = d_in, g.B = dY, g.ldb = d_out, g.C = part, g.ldc = d_out, g.bias = nullptr;
    g.M = d_in, g.N = d_out, g.K = n, g.alpha = 1.0f;
    const RowNormArgs r{X, dY, n, d_in, d_out, 1, rows};
    switch (xty_cfg(g.M, g.N, g.K, room)) {
        case GEMM_LARGE: return launch_xty_norms<ShapeLarge>(g, r, stream);
        case GEMM_WIDE: return launch_xty_norms<ShapeWide>(g, r, stream);
        case GEMM_SPLIT: return launch_xty_norms<ShapeSplit>(g, r, stream);
        case GEMM_MID: return launch_xty_norms<ShapeMid>(g, r, stream);
        case GEMM_COMPACT: return launch_xty_norms<ShapeCompact>(g, r, stream);
        case GEMM_FLAT: return launch_xty_norms<ShapeFlat>(g, r, stream);
        default: return launch_xty_norms<ShapeSmall>(g, r, stream);
    }
}

hipError_t launch_sketch_bf16(const bf16_t *A, bf16_t *out, int64_t n, int64_t d, int64_t k, int kind, SketchState st,
                              void *ws, hipStream_t stream, hipEvent_t ev_begin, hipEvent_t ev_end, int64_t d_other,
                              bool with_dbias, int64_t room) {
    EventPair pev(ev_begin, ev_end, stream);
    if (k <= kSmallK && (d_other == 0 || !small_pass_is_paired(n, d, d_other, k))) {  // bound by one pass over A: streaming kernel
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
    const SketchPlan p = with_dbias    ? plan_backward(n, d_other, d, k, kind, true, room).sketch
                         : d_other > 0 ? plan_pass(n, d, d_other, k, kind, room).sketch
                                       : plan_sketch(n, d, k, kind, true);
    const GemmArgs g = args_sketch(A, n, d, k, st, p, out, ws);
    hipError_t e = launch_sketch_plan(p, kind, g, stream);
    pev.done();
    if (e != hipSuccess || p.splits == 1) return e;
    return launch_reduce(ws, out, k, d, p.splits, stream);
}

hipError_t launch_forward_pair_bf16(const bf16_t *X, const bf16_t *W, const bf16_t *bias, bf16_t *Y, bf16_t *X_proj,
                                    int64_t n, int64_t d_in, int64_t d_out, int64_t k, int kind, SketchState st, void *ws, int64_t room,
                                    hipStream_t stream, hipEvent_t ev_begin, hipEvent_t ev_end) {
    const GemmArgs ga = args_nt(X, W, bias, Y, n, d_in, d_out);
    const PassPlan pass = plan_pass(n, d_in, d_out, k, kind, room);
    const SketchPlan &p = pass.sketch;
    const GemmArgs gb = args_sketch(X, n, d_in, k, st, p, X_proj, ws);
    EventPair pev(ev_begin, ev_end, stream);
    const hipError_t e = launch_pair_nt(pass, kind, ga, gb, stream);
    pev.done();
    if (e != hipSuccess || p.splits == 1) return e;
    return launch_reduce(ws, X_proj, k, d_in, p.splits, stream);
}

// Where the bias gradient goes in a backward pass that has the paired launch: into the launch of
// dW when that has room for it (dw_takes_colsum: dW is short and mostly latency); otherwise into the paired launch when dW runs on
// few_tile or the last round of the paired launch leaves at least 16 compute units idle (the sketch work-groups
// of that round run for long, and dY is being read there anyway; plan_backward sees to it where it
// can); otherwise behind the tiles of dW.  These share no launch where they are 256 x 256: column sums of their own then, or in the
// paired launch, unless it is made of such tiles too, on whose way into the chip column blocks can stand, and has no place for every
// block (57 passes: 2 % faster on average; without the last condition 3395 x 3056 -> 3960, k = 339: 212 -> 247 us).
bool backward_pair_takes_colsum_in(int64_t n, int64_t d_in, int64_t d_out, int64_t k, int kind, int64_t room) {
    if (!pass_pair_available(n, d_out, d_in, k)) return false;
    const int cfg = gemm_cfg(d_out, d_in, k);
    const PassPlan pass = plan_backward(n, d_in, d_out, k, kind, true, room);
    if (cfg == GEMM_LARGE) return pair_idle(pass) >= (pass.plain.cfg == GEMM_LARGE ? colsum_blocks(d_out, 2) : 16);
    return !dw_takes_colsum(d_in, d_out, k) && (cfg == GEMM_FEW || pair_idle(pass) >= 16);
}
bool backward_pair_takes_colsum(int64_t n, int64_t d_in, int64_t d_out, int64_t k, int kind) {
    return backward_pair_takes_colsum_in(n, d_in, d_out, k, kind, kMostSlices);
}

hipError_t launch_backward_pair_bf16(const bf16_t *dY, const bf16_t *W, bf16_t *dX, bf16_t *G, int64_t n, int64_t d_in,
                                     int64_t d_out, int64_t k, int kind, SketchState st, void *ws, int64_t room, hipStream_t stream,
                                     hipEvent_t ev_begin, hipEvent_t ev_end, bool with_dbias, bf16_t *dbias,
                                     bool accumulate_dbias) {
    const GemmArgs ga = args_nn(dY, W, dX, n, d_in, d_out);
    const PassPlan pass = plan_backward(n, d_in, d_out, k, kind, with_dbias, room);
    const SketchPlan &p = pass.sketch;
    const GemmArgs gb = args_sketch(dY, n, d_out, k, st, p, G, ws);
    const ColsumArgs gc{dY, dbias, n, d_out, accumulate_dbias ? 1 : 0, colsum_lpr(d_out, 2)};
    const ColsumArgs *gcp = dbias != nullptr ? &gc : nullptr;
    EventPair pev(ev_begin, ev_end, stream);
    const hipError_t e = launch_pair_nn(pass, kind, ga, gb, stream, gcp);
    pev.done();
    if (e != hipSuccess || p.splits == 1) return e;
    return launch_reduce(ws, G, k, d_out, p.splits, stream);
}

// ---- SORS kind: the plain product of a pass together with the strips of its sketch product (plan_sors).
bool sors_pair_available(int64_t n, int64_t d_sk, int64_t d_other, int64_t k) {
    return sors_fast_ok(n, d_sk) && plan_sors(n, d_sk, d_other, k).order != SORS_APART;
}

bool sors_strips_among_rounds(int64_t n, int64_t d_sk, int64_t d_other, int64_t k) {
    return sors_fast_ok(n, d_sk) && sors_among_rounds(n, d_sk, d_other, k) != SORS_APART;
}

static hipError_t launch_pass_sors(const GemmArgs &ga, bool row_indexed_b, const SorsArgs &gs, hipStream_t stream, hipEvent_t ev_begin,
                                   hipEvent_t ev_end) {
    const SorsPlan plan = plan_sors(gs.n, gs.d, ga.N, gs.k);
    EventPair pev(ev_begin, ev_end, stream);
    return launch_pair_sors(plan, row_indexed_b, ga, gs, stream);
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
