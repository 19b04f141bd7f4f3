// bf16 MFMA kernels of the RMM layer (gfx950): the five products of Algorithm 1,
//
//   Y      = X W^T          A = X  (K-contiguous rows)      B = W      (K-contiguous rows)
//   dX     = dY W           A = dY (K-contiguous rows)      B = W      (row-indexed)
//   X_proj = S^T X          A = P^T generated on chip       B = X      (row-indexed)
//   G      = S^T dY         A = P^T generated on chip       B = dY     (row-indexed)
//   dW     = G^T X_proj     A = G  (row-indexed)            B = X_proj (row-indexed)
//
// with C[M x N] = alpha * sum_kk A(m, kk) B(kk, n) on v_mfma_f32_32x32x16_bf16, fp32 accumulators.  An
// operand whose contraction index is its row index is read back from LDS with the transposing load
// ds_read_b64_tr_b16, which hands every lane four consecutive contraction elements of one column.
//
//   gemm_tile       Y, dX, dW and X^T dY on tiles from 64 x 64 to 256 x 256: memory straight into LDS, two to four
//                   stages of 64 contraction elements
//   few_tile        products with very few output tiles: the waves of a work-group share the contraction, no barriers
//   sketch_tile     sketch products with k > 64, and smaller ones in a paired launch, in the same kind of pipeline.  The sketch operand is never in
//                   memory: the work-group generates its tile of P^T into LDS (one 16-byte chunk = 8 consecutive
//                   tokens of one sketch column = one Philox-4x32-10 call for the Gaussian kind, one byte of a
//                   call's 128 sign bits for the Rademacher kind).  The 1/sqrt(k) of S = P/sqrt(k) is applied to
//                   the fp32 accumulator, so P is exact in bf16 for Rademacher and rounded once for Gaussian
//   sketch_smallk_kernel    the streaming kernel of small sketch sizes
//   reduce_partials_kernel  sums the partial results of token slices
//
// gemm_pair_kernel runs a plain product and the sketch product of a pass in one grid.
#pragma once
#include <type_traits>

#include "colsum.hpp"
#include "mfma_frag.hpp"
#include "row_norms.hpp"
#include "tile_range.hpp"

namespace rmm {

struct GemmArgs {
    const bf16_t *A;
    int64_t lda;
    const bf16_t *B;
    int64_t ldb;
    void *C;
    int64_t ldc;
    const bf16_t *bias;
    int64_t M, N, K;
    float alpha;
    int accumulate;        // bf16 output only: add the value C holds (in fp32, before the one rounding)
    SketchState st;
    int64_t k_chunk;       // sketch products: tokens per slice (multiple of 64)
    int slices, per_tail;  // sketch products: slices of k_chunk tokens of every tile; tiles whose last, short slice a further work-group takes
    int64_t split_stride;  // fp32 elements between the partial results of two slices
    int direct;            // partial-result kernels: there is one slice, write the bf16 result itself
};

namespace {

// Operands: rows along the contraction / rows across it (the contraction index is the row).
enum { A_KCONTIG = 0, A_MCONTIG = 1 };
enum { B_KCONTIG = 0, B_NCONTIG = 1 };
// Output: rounded to bf16 / fp32 partial result of a token slice (streaming sketch kernel) / no matrix at all, only
// the sum of squares of the tile (one double per work-group, C = double[work-groups]) / rounded to bf16, rows of any length.
enum { OUT_BF16 = 0, OUT_F32_PARTIAL = 1, OUT_SUMSQ = 2, OUT_BF16_ANY = 3 };

// Tiles of a plain product (gemm_tile): BM x BN outputs, WM x WN waves over the tile, WK groups of waves that take
// every other 16-deep contraction step, SA / SB LDS stages of the two operands, SP loads per wave and 16-deep step.
template <int BM_, int BN_, int WM_, int WN_, int WK_, int SA_, int SB_, int SP_>
struct TileShape {
    static constexpr int BM = BM_, BN = BN_, BK = 64, WM = WM_, WN = WN_, WK = WK_, SA = SA_, SB = SB_, SP = SP_;
    static constexpr int WAVES = WM * WN * WK, THREADS = 64 * WAVES;
    static constexpr int TM = BM / WM / 32, TN = BN / WN / 32;             // 32 x 32 MFMA tiles per wave
    static constexpr int A_ELEMS = BM * BK, B_ELEMS = BN * BK;             // of a stage
    static constexpr int A_LOADS = BM / 8 / WAVES, B_LOADS = BN / 8 / WAVES;  // 1 KB loads per wave and step
    static constexpr int LDS_BYTES = (SA * A_ELEMS + SB * B_ELEMS) * 2;
    static_assert(BM % (32 * WM) == 0 && BN % (32 * WN) == 0 && BM % (8 * WAVES) == 0 && BN % (8 * WAVES) == 0, "shares of a wave");
    static_assert(SB >= 2 && (SA == SB || SA == SB + 1) && SP * (4 / WK) >= A_LOADS + B_LOADS, "the loads of a step fit into it");
    static_assert(WK <= 2 && LDS_BYTES <= 160 * 1024, "LDS of a compute unit");
};
// (which product takes which: gemm_cfg and pair_plain in launch_plans.hpp)
typedef TileShape<256, 256, 2, 4, 1, 3, 2, 4> ShapeLarge;
typedef TileShape<128, 256, 2, 4, 1, 3, 3, 2> ShapeWide;
typedef TileShape<128, 128, 2, 2, 2, 3, 3, 3> ShapeSplit;
typedef TileShape<128, 128, 2, 4, 1, 3, 3, 1> ShapeMid;
typedef TileShape<128, 128, 2, 4, 1, 2, 2, 2> ShapeCompact;  // half of LDS: paired launches and X^T dY
typedef TileShape<64, 128, 2, 4, 1, 3, 3, 1> ShapeFlat;
typedef TileShape<64, 64, 2, 2, 1, 4, 4, 1> ShapeSmall;

// Tiles of a sketch product (sketch_tile).
template <int BM_, int BN_, int BK_, int WM_, int WN_, int WK_>
struct Shape {
    static constexpr int BM = BM_, BN = BN_, BK = BK_, WM = WM_, WN = WN_, WK = WK_;
    static constexpr int THREADS = 64 * WM * WN * WK;
};
typedef Shape<128, 512, 64, 1, 8, 1> ShapeSkWide;      // sketch products, tile generated into LDS;
typedef Shape<64, 512, 64, 1, 8, 1> ShapeSkWide64;     //   eight waves side by side: no two waves read the same B fragment
                                                       //   (64 instead of 80 KB of LDS reads per step)
typedef Shape<128, 384, 64, 2, 4, 1> ShapeSkMid;
typedef Shape<64, 384, 64, 2, 4, 1> ShapeSkMid64;
typedef Shape<128, 256, 64, 2, 4, 1> ShapeSkNarrow;
typedef Shape<64, 256, 64, 2, 4, 1> ShapeSkNarrow64;

// A Box-Muller pair of bf16 entries from one word of a Philox call: the radius, then the pair.
__device__ __forceinline__ float gauss_radius(uint32_t w) {
    const float u1 = fmaf((float)(w >> 16), 1.0f / 65536.0f, 1.0f / 131072.0f);  // (exact)
    return __builtin_amdgcn_sqrtf(-1.3862943611198906f * __builtin_amdgcn_logf(u1));  // -2 ln2 log2 u1
}
__device__ __forceinline__ bf16x2_t gauss_pair(uint32_t w, float rad) {
    const float u2 = (float)(w & 0xFFFFu) * (1.0f / 65536.0f);  // revolutions
    const f32x2_t z = {rad * __builtin_amdgcn_cosf(u2), rad * __builtin_amdgcn_sinf(u2)};
    return __builtin_convertvector(z, bf16x2_t);
}
// Eight unscaled Gaussian entries P[8*c0 .. 8*c0+7][j] as a bf16 MFMA operand.
__device__ __forceinline__ bf16x8_t gauss_operand(const SketchState &st, uint32_t c0, uint32_t j) {
    const Words4 r = philox4x32_10(c0, j, st.off0, st.off1, st.key0, st.key1);
    union {
        bf16x8_t v;
        bf16x2_t p[4];
    } out;
#pragma unroll
    for (int q = 0; q < 4; ++q) out.p[q] = gauss_pair(r.w[q], gauss_radius(r.w[q]));
    return out.v;
}

// Eight Rademacher entries from the lowest eight bits of `bits`.
__device__ __forceinline__ bf16x8_t radem_operand(uint32_t bits) {
    union {
        bf16x8_t v;
        uint32_t d[4];
    } out;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        out.d[q] = 0x3F803F80u | (((bits >> (2 * q)) & 1u) << 15) | (((bits >> (2 * q + 1)) & 1u) << 31);
    return out.v;
}
// The same for tokens t0 .. t0+7 (t0 a multiple of 8) of column j, given the four words of the call that covers
// tokens 128*(t0/128) .. +127.
__device__ __forceinline__ bf16x8_t radem_operand(const Words4 &r, uint32_t t0) {
    const uint32_t t = t0 & 127u;
    const uint32_t word = (t >> 5) == 0 ? r.w[0] : (t >> 5) == 1 ? r.w[1] : (t >> 5) == 2 ? r.w[2] : r.w[3];
    return radem_operand(word >> (t & 31u));
}

// The output tile of a wave.  The MFMA was issued with the operands swapped (B fragment first), so the
// accumulators hold C^T tiles: register v of lane l is C(l % 32, 8*(v/4) + 4*(l/32) + v%4)
// of its 32x32 tile, i.e. every lane owns four runs of four consecutive columns of one row.
// Storing that directly would touch 32 rows with 16 bytes each per instruction; instead every
// wave passes a strip of 32 rows x 128 bytes through a private piece of LDS (`stage`, kStripBytes) and
// writes it out with 16 bytes per lane, 8 lanes per row (full 128-byte lines).
// ANY: N is no multiple of 8, so that rows (and those 16 bytes) start anywhere; what of a chunk lies behind a row's end is not stored.
constexpr int kStripBytes = 32 * (128 + 16);
typedef u32x4_t u32x4_anywhere_t __attribute__((aligned(2)));
template <bool BF16, bool BIAS, bool ACCUMULATE, int TM, int TN, int WAVES_K, bool ANY = false>
__device__ __forceinline__ void write_tile(const GemmArgs &g, const f32x16_t (&acc)[TM][TN], char *stage, int64_t m0, int64_t n0,
                                           int wm, int wn, int kg, int lane, int slice = 0) {
    constexpr int WTM = 32 * TM, WTN = 32 * TN;
    constexpr int OWN = TM * TN / WAVES_K;               // tiles of a wave when WAVES_K groups share them
    constexpr int EB = BF16 ? 2 : 4;                     // bytes per output element
    constexpr int CW = 128 / EB;                         // columns per strip: 64 (bf16) or 32 (fp32)
    constexpr int TPS = CW / 32;                         // 32-column MFMA tiles per strip
    constexpr int PITCH = 128 + 16;                      // bytes per strip row in LDS
    static_assert(WAVES_K == 1 || (OWN % TPS == 0 && TN % TPS == 0), "no strip straddles the two groups' tiles");
    static_assert(PITCH * 32 == kStripBytes, "a wave's piece of LDS");
    const int r = lane & 31, h = lane >> 5;
    // The bias of this lane's columns does not depend on the row tile: fetched once, up front
    // (zeros where there is no bias or no column).
    constexpr bool MAY_HAVE_BIAS = BF16 && BIAS;  // Y = X W^T + 1 b^T only
    constexpr bool MAY_ACCUMULATE = BF16 && ACCUMULATE;                        // dW += G^T X_proj only
    uint2 bias_v[MAY_HAVE_BIAS ? TN : 1][4];
    if constexpr (MAY_HAVE_BIAS) {
#pragma unroll
        for (int b = 0; b < TN; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t col = n0 + wn * WTN + b * 32 + 8 * q + 4 * h;
                if constexpr (ANY) {
                    uint32_t e[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) e[u] = g.bias != nullptr && col + u < g.N ? g.bias[col + u] : 0u;
                    bias_v[b][q] = make_uint2(e[0] | e[1] << 16, e[2] | e[3] << 16);
                } else {
                    bias_v[b][q] = g.bias != nullptr && col < g.N ? *reinterpret_cast<const uint2 *>(g.bias + col) : make_uint2(0u, 0u);
                }
            }
    }
#pragma unroll
    for (int a = 0; a < TM; ++a) {
        const int64_t row0 = m0 + wm * WTM + a * 32;
#pragma unroll
        for (int b0 = 0; b0 < TN; b0 += TPS) {
            if (WAVES_K > 1 && (a * TN + b0) / OWN != kg) continue;  // the other group's tiles
            const int64_t col0 = n0 + wn * WTN + b0 * 32;
#pragma unroll
            for (int bb = 0; bb < TPS; ++bb) {
                if (b0 + bb >= TN) break;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float v[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) v[u] = acc[a][b0 + bb][4 * q + u];
                    const int c = bb * 32 + 8 * q + 4 * h;  // column inside the strip
                    if constexpr (BF16) {
#pragma unroll
                        for (int u = 0; u < 4; ++u) v[u] *= g.alpha;
                        if (MAY_ACCUMULATE && g.accumulate && row0 + r < g.M && col0 + c < g.N) {  // N is a multiple of 8
                            const uint2 cv = *reinterpret_cast<const uint2 *>(reinterpret_cast<const bf16_t *>(g.C) +
                                                                              (row0 + r) * g.ldc + col0 + c);
                            v[0] += __uint_as_float(cv.x << 16);
                            v[1] += __uint_as_float(cv.x & 0xFFFF0000u);
                            v[2] += __uint_as_float(cv.y << 16);
                            v[3] += __uint_as_float(cv.y & 0xFFFF0000u);
                        }
                        if (MAY_HAVE_BIAS && g.bias != nullptr) {  // (adding +0 would turn a -0 into +0: only where a bias exists)
                            const uint2 bv = bias_v[MAY_HAVE_BIAS ? b0 + bb : 0][q];
                            v[0] += __uint_as_float(bv.x << 16);
                            v[1] += __uint_as_float(bv.x & 0xFFFF0000u);
                            v[2] += __uint_as_float(bv.y << 16);
                            v[3] += __uint_as_float(bv.y & 0xFFFF0000u);
                        }
                        union {
                            bf16x2_t hh[2];
                            uint2 u;
                        } o;
                        o.hh[0] = __builtin_convertvector((f32x2_t){v[0], v[1]}, bf16x2_t);  // nearest even
                        o.hh[1] = __builtin_convertvector((f32x2_t){v[2], v[3]}, bf16x2_t);
                        *reinterpret_cast<uint2 *>(stage + r * PITCH + c * 2) = o.u;
                    } else {
                        *reinterpret_cast<float4 *>(stage + r * PITCH + c * 4) = make_float4(v[0], v[1], v[2], v[3]);
                    }
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            // read back: lane l takes 16 bytes: chunk (l % 8) of row (l / 8) + 8*i
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int rr = (lane >> 3) + 8 * i, ch = lane & 7;
                const uint4 d = *reinterpret_cast<const uint4 *>(stage + rr * PITCH + ch * 16);
                const int64_t row = row0 + rr, col = col0 + ch * (16 / EB);
                if (row >= g.M || col >= g.N || ch * (16 / EB) >= (TN - b0) * 32) continue;
                if constexpr (ANY) {
                    bf16_t *to = reinterpret_cast<bf16_t *>(g.C) + row * g.ldc + col;
                    if (col + 8 <= g.N) {
                        __builtin_nontemporal_store((u32x4_t){d.x, d.y, d.z, d.w}, reinterpret_cast<u32x4_anywhere_t *>(to));
                    } else {
                        const uint32_t w[4] = {d.x, d.y, d.z, d.w};
#pragma unroll
                        for (int u = 0; u < 8; ++u)
                            if (col + u < g.N) to[u] = (bf16_t)(w[u / 2] >> (u % 2 * 16));
                    }
                } else if constexpr (BF16)
                    // non-temporal: all work-groups of a round write their tiles at the same time, and
                    // nothing reads them before the kernel ends
                    __builtin_nontemporal_store((u32x4_t){d.x, d.y, d.z, d.w},
                                                reinterpret_cast<u32x4_t *>(reinterpret_cast<bf16_t *>(g.C) + row * g.ldc + col));
                else
                    *reinterpret_cast<uint4 *>(reinterpret_cast<float *>(g.C) +
                                               (int64_t)slice * g.split_stride + row * g.ldc + col) = d;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    }
}

// ---------------------------------------------------------------------------------------------
// The plain products.  Memory -> LDS without registers in between (buffer_load ... lds, 16 bytes per lane, a wave's
// 64 lanes = 1 KB of consecutive LDS), in steps of 64 contraction elements: whole 128-byte lines of K-contiguous
// rows.  What bounds it is that path: a compute unit takes at most 64 bytes per clock from L2, about 40 where the whole
// chip pulls 256 x 256 tiles (a loop of these loads alone, 64 KB in flight), against the 32 its MFMAs need with such
// tiles and the 64 with 128 x 128; and that the first load of a line waits for HBM.  So
//   - the tile is as large as the number of tiles allows;
//   - the loads of a step are spread between the MFMAs of two 16-deep steps, SP per wave and 16-deep step, instead of
//     being issued in one burst behind the barrier, where the MFMAs behind them in the instruction stream wait until the
//     burst is taken (256 x 256, 16384 x 4096 -> 1024: 125 -> 113 us; 128 x 128, 4096 x 3072 -> 768: 28 -> 26);
//   - the operand that streams (A: tokens) gets one LDS stage more than the weights where all of LDS is one tile's (256 x
//     256: 113 -> 108 us), and smaller tiles have three or four stages.
// Every instruction of a step has its place: an MFMA, then the LDS reads and loads that go with it (sched_barrier);
// left to itself the compiler bunches the reads in front of their use.
//
// LDS is laid out by the load, so what keeps bank conflicts away is which chunk a lane asks for: rows of 64 contraction
// elements hold chunk c at kchunk_pos, rows of columns at col_chunk.

// One wave's load of 1 KB into LDS from byte `to` on, 16 bytes from `off` + `soff` per lane.  The compiler does
// not see that it writes LDS (it would wait for it before every LDS read): the explicit waits and barriers order them.
__device__ __forceinline__ void load_to_lds(u32x4_t rsrc, uint32_t to, uint32_t off, uint32_t soff) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(to), "v"(off), "s"(rsrc), "s"(soff) : "m0");
}
// The same from `off`.
__device__ __forceinline__ void load_to_lds(u32x4_t rsrc, uint32_t to, uint32_t off) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(to), "v"(off), "s"(rsrc) : "m0");
}
// Waits until at most N of this wave's loads are outstanding.
template <int N>
__device__ __forceinline__ void wait_for_loads() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// A descriptor of `rows` rows of pitch ld from `base` on.  (The same in every lane; saying so keeps it in scalar registers.)
__device__ __forceinline__ u32x4_t rows_descriptor(const bf16_t *base, int64_t ld, int64_t rows) {
    const uint64_t at = reinterpret_cast<uint64_t>(base);
    return (u32x4_t){(uint32_t)__builtin_amdgcn_readfirstlane((int)at), (uint32_t)__builtin_amdgcn_readfirstlane((int)(at >> 32)),
                     (uint32_t)__builtin_amdgcn_readfirstlane((int)((rows > 0 ? rows : 0) * ld * 2)), 0x00020000u};
}
// The wait states between a vector instruction that writes a scalar register (a readfirstlane, a spilled one that comes back) and a
// load that reads it: the compiler does not look for them in front of load_to_lds.  What a step of a K-contiguous operand writes (the range
// of its descriptor, the offset along its rows) is scalar instructions, which need none, and is not settled: twenty clocks a step and
// operand, 64 x 64 tiles of Y 5 % (1024 x 1024 -> 512 5.8 and 6.1 us).  That the compiler brings none of it back from a vector register too
// close to a load is looked for in the built library (tests/test_load_hazards.py).
__device__ __forceinline__ void settle(u32x4_t &descriptor) { asm volatile("s_nop 4" : "+s"(descriptor)); }
// The steps of 64 contraction elements in the order in which a work-group takes them: from `start` on and around.  What a request
// needs is prepared one step ahead, between MFMAs, from what the one before it needed, in scalar registers and mostly 32 bits.  Made
// anew, with products of 64 bits, selects and a way through the vector unit, it was 45 of the 62 scalar instructions of a step of
// X^T dY, in one piece between two MFMAs, for both waves of a SIMD at once (it is 22 of 39; 4096 x 768 x 3072: a step of 64 0.48 ->
// 0.42 us, the monitors 37.3 -> 32.7; dX of 192 128 x 128 tiles, K-contiguous Y: 49 -> 42 and 35 -> 30 a step; whole steps 1.00 to 1.06,
// 16384 x 1024 -> 4096 567 -> 556).  A scalar instruction costs a wave about as much of its time as a vector one.
struct Walk {
    int steps, to_wrap, todo;  // steps until the walk is at the end of the contraction, and steps that are left
    uint32_t soff;             // of the step that is next, in bytes along a K-contiguous row
    __device__ __forceinline__ void init(int kk, int start) {
        steps = todo = (kk + 63) / 64, to_wrap = __builtin_amdgcn_readfirstlane(steps - start), soff = (uint32_t)(steps - to_wrap) * 128u;
    }
};
// 64 rows a step of a row-indexed operand.
struct StepRows {
    uint64_t base, next;  // first row of the contraction, of the next step
    uint32_t step_bytes, last_bytes;
    __device__ __forceinline__ void init(const bf16_t *first, int64_t ld, int kk, const Walk &w) {  // (rows below 2^22 elements)
        step_bytes = 128u * (uint32_t)ld, last_bytes = 2u * (uint32_t)ld * (uint32_t)(kk - (w.steps - 1) * 64);
        base = reinterpret_cast<uint64_t>(first), next = base + (uint64_t)(uint32_t)(w.steps - w.to_wrap) * step_bytes;
    }
    // The descriptor of the next step (past the end: of none, a load writes zeros).
    __device__ __forceinline__ u32x4_t descriptor(bool last, bool live) {
        const uint64_t at = next, behind = next + step_bytes;
        const uint32_t bytes = last ? last_bytes : step_bytes;
        next = last ? base : behind;
        return (u32x4_t){(uint32_t)at, (uint32_t)(at >> 32), live ? bytes : 0u, 0x00020000u};
    }
};
// Prepares the next step of a walk for what takes it.
template <typename... Operands>
__device__ __forceinline__ void prepare_step(Walk &w, Operands &...operands) {
    const uint32_t along = w.soff + 128u;
    const bool last = w.to_wrap == 1, live = w.todo > 0;
    (operands.prepare(w, last, live), ...);
    w.to_wrap = last ? w.steps : w.to_wrap - 1, w.soff = last ? 0u : along, --w.todo;
}

// Rows of C columns, contraction row k: chunk c (eight columns) sits at position col_chunk(k, c) and the other way round.
// The four rows of a transposing read (k, k + 1, k + 2, k + 3) then fall on different 64 bytes of the banks.
template <int C>
__device__ __forceinline__ int col_chunk(int k, int chunk) {
    return chunk ^ (C >= 128 ? (k & 3) << 2 : (k & 2) << 1);
}
// (see frag_transposed) from rows of C columns placed like that
template <int C>
__device__ __forceinline__ bf16x8_t frag_columns(const bf16_t *tile, int col0, int kk0, int lane) {
    const int blk = lane >> 4, i = lane & 15, k = kk0 + ((blk >> 1) << 3) + (i >> 2), col = col0 + ((blk & 1) << 4) + ((i & 3) << 2);
    const bf16_t *p = tile + k * C + (col_chunk<C>(k, col >> 3) << 3) + (col & 7);
    typedef __attribute__((address_space(3))) s16x4_t *lds_ptr_t;
    const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(p));
    const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(p + 4 * C));  // (row k + 4: same k % 4)
    union {
        s16x8_t s;
        bf16x8_t v;
    } out;
    out.s = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return out.v;
}

// One operand of a tile on its way into LDS: E rows of 64 contraction elements (KROWS) or 64 contraction rows of E
// columns, J loads of 1 KB per wave.  An offset at or beyond the descriptor's byte range writes zeros without touching
// memory, so edges and tails need no branches (a chunk that must read as zero gets the offset 2^31).  A descriptor spans
// only what the work-group reads of the operand, so that 32-bit offsets suffice for operands of any size: the tile's rows,
// fixed for the kernel, or the 64 contraction rows of a step.
template <int E, int J, bool KROWS>
struct OperandLoads {
    static constexpr uint32_t OOB = 0x80000000u;
    uint32_t off[J], beyond[KROWS ? J : 1];  // of a step; all ones where the last one of the contraction has nothing
    StepRows rows;
    uint32_t range;                            // K-contiguous: bytes of the tile's rows
    u32x4_t ready, rsrc;                       // descriptors: of the step that is next, of the one that is being requested;
    uint32_t ready_soff, ready_oob, soff, oob; //   where it is along the rows, and what the chunks beyond a last step get or'ed to their offsets
    uint32_t to;
    __device__ __forceinline__ void init(const bf16_t *operand, int64_t ld, int64_t row0, int64_t count, int kk, const Walk &w, int wave, int lane) {
#pragma unroll
        for (int j = 0; j < J; ++j) {
            if constexpr (KROWS) {
                const int row = (wave * J + j) * 8 + (lane >> 3), chunk = kchunk_pos<64>(row, lane & 7);
                off[j] = row0 + row < count ? (uint32_t)((row * ld + chunk * 8) * 2) : OOB;
                beyond[j] = chunk * 8 < kk - (w.steps - 1) * 64 ? 0u : 0xFFFFFFFFu;
            } else {
                const int c = (wave * J + j) * 64 + lane, k = c / (E / 8), col = col_chunk<E>(k, c % (E / 8)) * 8;
                off[j] = row0 + col < count ? (uint32_t)((k * ld + row0 + col) * 2) : OOB;
            }
        }
        if constexpr (KROWS)
            rsrc = rows_descriptor(operand + row0 * ld, ld, min((int64_t)E, count - row0)), settle(rsrc), range = rsrc[2];
        else
            rows.init(operand, ld, kk, w);
    }
    // The step that is next (prepare_step; past the end: zeros).
    __device__ __forceinline__ void prepare(const Walk &w, bool last, bool live) {
        ready_soff = KROWS ? w.soff : 0u;
        if constexpr (KROWS) {
            ready_oob = last ? OOB : 0u, ready[2] = live ? range : 0u;
        } else {
            ready = rows.descriptor(last, live);
        }
    }
    // The step that was prepared goes to LDS byte `to_` (of this wave's share).
    __device__ __forceinline__ void begin(uint32_t to_) {
        to = to_, soff = ready_soff;
        if constexpr (KROWS) {
            rsrc[2] = ready[2], oob = ready_oob;
        } else {
            rsrc = ready, settle(rsrc);
        }
    }
    __device__ __forceinline__ void load(int j) const {
        if constexpr (KROWS)
            load_to_lds(rsrc, to + j * 1024, off[j] | (oob & beyond[j]), soff);
        else
            load_to_lds(rsrc, to + j * 1024, off[j]);
    }
};
// First row and column of output tile number `tile`: bands of 8 tile rows, column by column.
template <int BM, int BN>
__device__ __forceinline__ void tile_origin(uint32_t tile, uint32_t tiles_m, uint32_t tiles_n, int64_t &m0, int64_t &n0) {
    constexpr uint32_t GROUP_M = 8;
    const uint32_t band = tile / (GROUP_M * tiles_n), in_band = tile - band * (GROUP_M * tiles_n);
    const uint32_t band_rows = min(GROUP_M, tiles_m - band * GROUP_M), col = in_band / band_rows;
    m0 = (int64_t)(band * GROUP_M + in_band - col * band_rows) * BM, n0 = (int64_t)col * BN;
}

// One work-group's share of a product: output tile number `block` of `blocks`.  `lds` holds S::LDS_BYTES bytes.
template <typename S, int AMODE, int BMODE, int OUT>
__device__ __forceinline__ void gemm_tile(const GemmArgs &g, bf16_t *lds, int64_t block, int64_t blocks) {
    constexpr int BM = S::BM, BN = S::BN, BK = S::BK, SA = S::SA, SB = S::SB, SP = S::SP, TM = S::TM, TN = S::TN;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Wave w works on the (wm, wn) part of the tile and, of every 16-deep contraction step s, on those with s % WK == kg.
    const int kg = wave / (S::WM * S::WN), wmn = wave % (S::WM * S::WN), wm = wmn / S::WN, wn = wmn % S::WN;
    // Tile order.  Work-groups are dealt round-robin to the 8 XCDs (each with its own L2), so first
    // renumber them such that one XCD owns a contiguous run of positions; then walk the tile grid
    // in bands of GROUP_M tile rows, column by column, so that the work-groups resident on one XCD
    // at the same time form a compact block that shares A row blocks and B column blocks in L2.
    // (In 32 bits: a grid has fewer than 2^31 work-groups, and five divisions of 64 bits stood in front of the first load: a step of
    // 1277 x 344 -> 344, k = 64, 31.3 -> 30.6 us, of 16384 x 1024 -> 4096 559 -> 557.)
    const uint32_t tiles_m = (uint32_t)((g.M + BM - 1) / BM), tiles_n = (uint32_t)((g.N + BN - 1) / BN);
    uint32_t tile;
    {
        const uint32_t per = (uint32_t)blocks / 8, rem = (uint32_t)blocks % 8, x = (uint32_t)block % 8, r = (uint32_t)block / 8;
        tile = x * per + (x < rem ? x : rem) + r;   // XCD x owns `per` (+1 for the first `rem`) consecutive positions
    }
    int64_t m0, n0;
    tile_origin<BM, BN>(tile, tiles_m, tiles_n, m0, n0);
    const int kk = (int)g.K, steps = (kk + BK - 1) / BK;
    // Work-groups walk the contraction from different starting steps (and wrap around): with a
    // power-of-two row pitch all rows of a tile fall on the same one or two L2 channels, and the
    // rotation spreads concurrently running work-groups over the channels.
    const int stagger = (int)((AMODE == A_KCONTIG && BMODE == B_KCONTIG ? start_of_place(m0, n0, g.N) : start_of_tile(tile)) % (uint32_t)steps);

    constexpr int JA = S::A_LOADS, JB = S::B_LOADS, LOADS = JA + JB;
    OperandLoads<BM, JA, AMODE == A_KCONTIG> la;
    OperandLoads<BN, JB, BMODE == B_KCONTIG> lb;
    Walk walk, walk_a;  // (with as many stages of A as of B one serves both)
    walk.init(kk, stagger), walk_a.init(kk, stagger);
    la.init(g.A, g.lda, m0, g.M, kk, walk, wave, lane);
    lb.init(g.B, g.ldb, n0, g.N, kk, walk, wave, lane);
    typedef __attribute__((address_space(3))) bf16_t *lds_ptr_t;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr_t)lds;
    const uint32_t share_a = lds0 + (uint32_t)(wave * JA * 1024), share_b = lds0 + (uint32_t)(SA * S::A_ELEMS * 2 + wave * JB * 1024);
    auto begin_a = [&](int stage) { la.begin(share_a + (uint32_t)(stage * S::A_ELEMS * 2)); };
    auto begin_b = [&](int stage) { lb.begin(share_b + (uint32_t)(stage * S::B_ELEMS * 2)); };
    auto load = [&](int i) {  // load i of a step: B's come first (with SA > SB they are waited for first)
        if (i < JB)
            lb.load(i);
        else if (i < LOADS)
            la.load(i - JB);
    };

    f32x16_t acc[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.0f;
    struct Frags {
        bf16x8_t a[TM], b[TN];
    };
    constexpr int FRAGS = TM + TN, MFMAS = TM * TN, KS = BK / 16 / S::WK;
    static_assert(KS % 2 == 0, "the first fragments of a step are always in f[0]");
    // Fragment i of this wave's ks-th 16-deep step of the tile in stages (sa, sb).
    auto read = [&](Frags &f, int sa, int sb, int ks, int i) {
        const int k0 = (ks * S::WK + kg) * 16;
        if (i < TN) {
            const bf16_t *Bs = lds + SA * S::A_ELEMS + sb * S::B_ELEMS;
            const int col0 = wn * (BN / S::WN) + i * 32;
            if constexpr (BMODE == B_KCONTIG)
                f.b[i] = frag_kcontig<BK>(Bs, col0, k0, lane);
            else
                f.b[i] = frag_columns<BN>(Bs, col0, k0, lane);
        } else {
            const bf16_t *As = lds + sa * S::A_ELEMS;
            const int row0 = wm * (BM / S::WM) + (i - TN) * 32;
            if constexpr (AMODE == A_KCONTIG)
                f.a[i - TN] = frag_kcontig<BK>(As, row0, k0, lane);
            else
                f.a[i - TN] = frag_columns<BM>(As, row0, k0, lane);
        }
    };
    // One 16-deep step: multiplies `now`, reads the fragments of the one behind it and issues SP loads from load l0 on.
    auto sixteen = [&](const Frags &now, Frags &next, int sa, int sb, int ks, int l0) {
#pragma unroll
        for (int i = 0; i < MFMAS; ++i) {
            const int a = i / TN, b = i % TN;
            acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(now.b[b], now.a[a], acc[a][b], 0, 0, 0);
#pragma unroll
            for (int r = i * FRAGS / MFMAS; r < (i + 1) * FRAGS / MFMAS; ++r) read(next, sa, sb, ks, r);
#pragma unroll
            for (int r = i * SP / MFMAS; r < (i + 1) * SP / MFMAS; ++r) load(l0 + r);
            const int slot = l0 / SP * MFMAS - MFMAS + i;  // behind the barrier's step: what the next begin needs, away from the barrier
            if constexpr (SA == SB) {
                if (l0 > 0 && slot == (KS - 1) * MFMAS / 2) prepare_step(walk, la, lb);
            } else {
                if (l0 > 0 && slot == 0) prepare_step(walk_a, la);
                if (l0 > 0 && slot == (KS - 1) * MFMAS / 2) prepare_step(walk, lb);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // Step t of A is in stage t % SA, of B in stage t % SB.  The one barrier of a step stands in front of its last 16-deep
    // step: by then every wave holds that one's fragments in registers, so the stages can be overwritten (step t + SA of A
    // and t + SB of B are requested from here on), and the data of step t + 1 has been waited for, so its first fragments
    // are read under the MFMAs of the last 16-deep step: no step begins by waiting for LDS.  Steps past the end are
    // requested as zeros, which keeps the number of outstanding loads the same.
    constexpr int OUTSTANDING = (SB - 2) * LOADS + (SA > SB ? JA : 0);  // behind the loads of step t + 1
    Frags f[2];
#pragma unroll
    for (int s = 0; s < SA - 1; ++s) {
        if constexpr (SA == SB)
            prepare_step(walk, la, lb);
        else
            prepare_step(walk_a, la);
        begin_a(s);
#pragma unroll
        for (int j = 0; j < JA; ++j) la.load(j);
        if (s < SB - 1) {
            if constexpr (SA != SB) prepare_step(walk, lb);
            begin_b(s);
#pragma unroll
            for (int j = 0; j < JB; ++j) lb.load(j);
        }
    }
    wait_for_loads<(SA - 2) * JA + (SB - 2) * JB>();
    __syncthreads();
#pragma unroll
    for (int i = 0; i < FRAGS; ++i) read(f[0], 0, 0, 0, i);
    if constexpr (SA == SB)
        prepare_step(walk, la, lb);
    else
        prepare_step(walk_a, la), prepare_step(walk, lb);
    begin_b(SB - 1), begin_a(SA - 1);
#pragma unroll
    for (int i = 0; i < SP; ++i) load(i);
    auto one_step = [&](int sa, int sb) __attribute__((always_inline)) {
        const int next_a = sa == SA - 1 ? 0 : sa + 1, next_b = sb == SB - 1 ? 0 : sb + 1;
#pragma unroll
        for (int ks = 0; ks < KS - 1; ++ks) sixteen(f[ks & 1], f[(ks + 1) & 1], sa, sb, ks + 1, (ks + 1) * SP);
        wait_for_loads<OUTSTANDING>();
        __syncthreads();
        begin_b(sb), begin_a(sa);
        sixteen(f[1], f[0], next_a, next_b, 0, 0);  // (past the end: zeros, not used)
    };
    if constexpr (SA == SB) {
        // The stages one after the other: their places in LDS are offsets of the instructions.
        int t = 0;
        for (; t + SA <= steps; t += SA)
#pragma unroll
            for (int s = 0; s < SA; ++s) one_step(s, s);
#pragma unroll
        for (int s = 0; s < SA - 1; ++s)
            if (t + s < steps) one_step(s, s);
    } else {
        int sa = 0, sb = 0;
        for (int t = 0; t < steps; ++t) {
            one_step(sa, sb);
            sa = sa == SA - 1 ? 0 : sa + 1, sb = sb == SB - 1 ? 0 : sb + 1;
        }
    }
    wait_for_loads<0>();
    __syncthreads();  // LDS is free

    // Two wave groups that split the contraction each end up owning half of the 32x32 tiles of
    // their (identical) wave tile: a group parks the tiles the other one owns in LDS, 16 bytes per
    // lane and run with consecutive lanes consecutive, in rounds that fit the LDS, and adds what
    // the other group parked for it.  Both groups then write their halves.
    constexpr int P = TM * TN;       // tiles per wave, numbered a * TN + b
    constexpr int OWN = P / S::WK;  // group kg owns tiles kg*OWN .. kg*OWN + OWN - 1
    if constexpr (S::WK == 2) {
        static_assert(P % 2 == 0, "an even number of tiles per wave");
        constexpr int CH_MAX = S::LDS_BYTES / (64 * S::THREADS);  // tiles per thread and round that fit
        static_assert(CH_MAX >= 1, "one tile per thread fits in LDS");
        constexpr int CH = OWN < CH_MAX ? OWN : CH_MAX;
        float4 *park = reinterpret_cast<float4 *>(lds);
        constexpr int GROUP_THREADS = S::THREADS / 2;
        const int partner = kg == 0 ? tid + GROUP_THREADS : tid - GROUP_THREADS;
        // `from` is a literal at every call, so all accumulator indices are static after unrolling.
        auto park_tiles = [&](auto from, int c0) {
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const int p = decltype(from)::value + c0 + c;
                if (c0 + c < OWN) {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        park[(c * 4 + q) * S::THREADS + tid] =
                            make_float4(acc[p / TN][p % TN][4 * q], acc[p / TN][p % TN][4 * q + 1], acc[p / TN][p % TN][4 * q + 2],
                                        acc[p / TN][p % TN][4 * q + 3]);
                }
            }
        };
        auto add_tiles = [&](auto from, int c0) {
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const int p = decltype(from)::value + c0 + c;
                if (c0 + c < OWN) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const float4 pv = park[(c * 4 + q) * S::THREADS + partner];
                        acc[p / TN][p % TN][4 * q] += pv.x, acc[p / TN][p % TN][4 * q + 1] += pv.y;
                        acc[p / TN][p % TN][4 * q + 2] += pv.z, acc[p / TN][p % TN][4 * q + 3] += pv.w;
                    }
                }
            }
        };
        using Zero = std::integral_constant<int, 0>;
        using Half = std::integral_constant<int, OWN>;
#pragma unroll
        for (int c0 = 0; c0 < OWN; c0 += CH) {
            if (kg == 0)
                park_tiles(Half(), c0);  // group 0 gives away the upper half
            else
                park_tiles(Zero(), c0);
            __syncthreads();
            if (kg == 0)
                add_tiles(Zero(), c0);
            else
                add_tiles(Half(), c0);
            __syncthreads();
        }
    }
    if constexpr (OUT == OUT_SUMSQ) {
        // Squared Frobenius norm of the tile: rows and columns beyond the matrix were loaded as
        // zeros, so they add nothing.  Per-lane sums, wave reduction, then the waves' sums in fp64.
        float sq = 0.0f;
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
            for (int b = 0; b < TN; ++b) {
                if (S::WK > 1 && (a * TN + b) / OWN != kg) continue;  // the other group's tiles
#pragma unroll
                for (int v = 0; v < 16; ++v) sq += acc[a][b][v] * acc[a][b][v];
            }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) sq += __shfl_xor(sq, off, 64);
        double *red = reinterpret_cast<double *>(lds);
        if (lane == 0) red[wave] = (double)sq;
        __syncthreads();
        if (tid == 0) {
            double t = 0.0;
#pragma unroll
            for (int w = 0; w < S::WAVES; ++w) t += red[w];
            reinterpret_cast<double *>(g.C)[block] = t;
        }
    } else {
        static_assert(S::WAVES * kStripBytes <= S::LDS_BYTES, "staging area fits in LDS");
        char *strip = reinterpret_cast<char *>(lds) + wave * kStripBytes;
        write_tile<true, AMODE == A_KCONTIG && BMODE == B_KCONTIG, AMODE == A_MCONTIG, TM, TN, S::WK, OUT == OUT_BF16_ANY>(g, acc, strip, m0, n0, wm, wn, kg, lane);
    }
}

// ---------------------------------------------------------------------------------------------
// Products with few output tiles (short requests, narrow layers, dW of a base layer): what bounds them
// is the chain of loads, LDS and barriers along the contraction, not bandwidth or MFMA rate.  So a
// work-group takes an E x E tile, its eight waves an eighth of the contraction each, and a
// wave walks its share without a barrier, 64 contraction elements per step through a piece of LDS of its
// own (128-byte lines from memory, the MFMA's layout out of LDS), with the next two steps in flight.  The
// eight partial tiles meet once, in LDS, in wave order.
// 24 x 768 -> 3072: kernel 8.3 us with 64 x 64 tiles and a barrier every 32 elements, call 9.5 -> 5.2 us.
constexpr int kFewThreads = 512;
struct FewTile {
    static constexpr int E = 32, BK = 64;           // edge of the tile; contraction elements per step of a wave
    static constexpr int LOADS = E * BK / 8 / 64;   // 16-byte loads per lane, operand and step
    static constexpr int PATCH = BK * E;            // elements of a wave's piece of one operand
    static constexpr int LDS_BYTES = 8 * 2 * PATCH * 2;
    static_assert(LDS_BYTES >= 8 * E * E * 4, "room for the partial tiles");
};

template <int AMODE, int BMODE, bool SINGLE>
__device__ __forceinline__ void few_tile(const GemmArgs &g, unsigned char *lds, int64_t block, int64_t blocks) {
    typedef FewTile F;
    constexpr int E = F::E, BK = F::BK, L = F::LOADS;
    constexpr bool A_K = AMODE == A_KCONTIG, B_K = BMODE == B_KCONTIG;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t tiles_m = (uint32_t)((g.M + E - 1) / E);
    uint32_t tile = (uint32_t)block;
    {
        const uint32_t per = (uint32_t)blocks / 8, rem = (uint32_t)blocks % 8, x = tile % 8, r = tile / 8;
        tile = x * per + (x < rem ? x : rem) + r;  // an XCD takes neighbouring tiles: same columns, other rows
    }
    const uint32_t tile_n = tile / tiles_m;
    const int64_t m0 = (int64_t)(tile - tile_n * tiles_m) * E, n0 = (int64_t)tile_n * E;
    const int64_t steps = (g.K + 15) / 16, share = (steps + 7) / 8;
    const int64_t k_begin = wave * share * 16;
    const int k_len = (int)max((int64_t)0, min(g.K, k_begin + share * 16) - k_begin);  // this wave's contraction elements

    constexpr uint32_t OOB = 0x80000000u;
    auto range = [](const bf16_t *base, int64_t elems) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(base), (short)0,
                                                 __builtin_amdgcn_readfirstlane((int)(elems > 0 ? elems * 2 : 0)), 0x00020000);
    };
    // K-contiguous: load u of lane l takes chunk l % 8 (eight elements) of row 8u + l / 8.
    // Row-indexed:  load u of lane l takes chunk l % (E/8) of contraction row (512/E)u + l / (E/8).
    constexpr int CPR = E / 8;
    const int kr = lane >> 3, kc = (lane & 7) * 8, nr = lane / CPR, nc = lane % CPR * 8;
    uint32_t a_off[L], b_off[L];
    int a_at[L], b_at[L];
#pragma unroll
    for (int u = 0; u < L; ++u) {
        const int rk = 8 * u + kr, rn = 64 / CPR * u + nr;
        const int at_k = rk * BK + kchunk_pos<BK>(rk, lane & 7) * 8, at_n = rn * E + nc;
        a_off[u] = A_K ? (m0 + rk < g.M ? (uint32_t)((rk * g.lda + kc) * 2) : OOB) : (m0 + nc < g.M ? (uint32_t)((rn * g.lda + nc) * 2) : OOB);
        b_off[u] = B_K ? (n0 + rk < g.N ? (uint32_t)((rk * g.ldb + kc) * 2) : OOB) : (n0 + nc < g.N ? (uint32_t)((rn * g.ldb + nc) * 2) : OOB);
        a_at[u] = A_K ? at_k : at_n, b_at[u] = B_K ? at_k : at_n;
    }
    bf16_t *patch_a = reinterpret_cast<bf16_t *>(lds) + wave * 2 * F::PATCH, *patch_b = patch_a + F::PATCH;

    struct Step {
        u32x4_t a[L], b[L];
    };
    // Elements k0 .. k0 + BK - 1 of this wave's share; what lies beyond it reads as zero.
    auto request = [&](Step &q, int k0) {
        const int left = max(0, k_len - k0);
        // (rows m0 .. from element k_begin + k0 on / contraction rows k_begin + k0 .. of columns m0 ..)
        const __amdgpu_buffer_rsrc_t ra =
            A_K ? range(g.A + m0 * g.lda + k_begin + k0, left > 0 ? (min((int64_t)E, g.M - m0) - 1) * g.lda + left : 0)
                : range(g.A + (k_begin + k0) * g.lda + m0, left > 0 ? (min(left, BK) - 1) * g.lda + (g.M - m0) : 0);
        const __amdgpu_buffer_rsrc_t rb =
            B_K ? range(g.B + n0 * g.ldb + k_begin + k0, left > 0 ? (min((int64_t)E, g.N - n0) - 1) * g.ldb + left : 0)
                : range(g.B + (k_begin + k0) * g.ldb + n0, left > 0 ? (min(left, BK) - 1) * g.ldb + (g.N - n0) : 0);
        const bool ok_k = kc < left;
#pragma unroll
        for (int u = 0; u < L; ++u) {
            q.a[u] = __builtin_amdgcn_raw_buffer_load_b128(ra, !A_K || ok_k ? a_off[u] : OOB, 0, 0);
            q.b[u] = __builtin_amdgcn_raw_buffer_load_b128(rb, !B_K || ok_k ? b_off[u] : OOB, 0, 0);
        }
    };
    f32x16_t acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
    auto wave_sync = [] {  // orders a wave's own LDS accesses (LDS serves a wave's instructions in order)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    auto multiply = [&](const Step &q) {
        wave_sync();  // the step before has been read
#pragma unroll
        for (int u = 0; u < L; ++u) {
            *reinterpret_cast<u32x4_t *>(patch_a + a_at[u]) = q.a[u];
            *reinterpret_cast<u32x4_t *>(patch_b + b_at[u]) = q.b[u];
        }
        wave_sync();
#pragma unroll
        for (int u = 0; u < BK / 16; ++u) {
            const bf16x8_t a = A_K ? frag_kcontig<BK>(patch_a, 0, 16 * u, lane) : frag_transposed(patch_a, E, 0, 16 * u, lane);
            const bf16x8_t b = B_K ? frag_kcontig<BK>(patch_b, 0, 16 * u, lane) : frag_transposed(patch_b, E, 0, 16 * u, lane);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
        }
    };
    if constexpr (SINGLE) {  // a contraction of at most 8 * BK: nothing to prefetch
        Step q;
        request(q, 0);
        multiply(q);
    } else {
        Step q[2];
        request(q[0], 0);
        request(q[1], BK);
        for (int k0 = 0; k0 < k_len; k0 += 2 * BK) {
            multiply(q[0]);
            request(q[0], k0 + 2 * BK);
            multiply(q[1]);
            request(q[1], k0 + 3 * BK);
        }
    }
    __syncthreads();  // the pieces are free
    // Register v of lane l is C(8*(v/4) + 4*(l/32) + v%4, l % 32) of a 32 x 32 tile.
    float *red = reinterpret_cast<float *>(lds);
#pragma unroll
    for (int v = 0; v < 16; ++v) red[wave * 1024 + v * 64 + lane] = acc[v];
    __syncthreads();
    // A thread finishes two neighbouring columns of rows tid / (E/2), ...
    const int r = tid / (E / 2), c = tid % (E / 2) * 2;
    const int64_t col = n0 + c;
    float b0 = 0.0f, b1 = 0.0f;
    if (g.bias != nullptr && col < g.N) {
        const uint32_t o = *reinterpret_cast<const uint32_t *>(g.bias + col);
        b0 = __uint_as_float(o << 16), b1 = __uint_as_float(o & 0xFFFF0000u);
    }
    const int at = ((r >> 3) * 4 + (r & 3)) * 64 + ((r >> 2) & 1) * 32 + c;
    float x0 = 0.0f, x1 = 0.0f;
#pragma unroll
    for (int w = 0; w < 8; ++w) {
        const float2 p = *reinterpret_cast<const float2 *>(red + w * 1024 + at);
        x0 += p.x, x1 += p.y;
    }
    const int64_t row = m0 + r;
    if (row >= g.M || col >= g.N) return;  // N is a multiple of 8
    bf16_t *out = reinterpret_cast<bf16_t *>(g.C) + row * g.ldc + col;
    x0 *= g.alpha, x1 *= g.alpha;
    if (g.accumulate) {
        const uint32_t o = *reinterpret_cast<const uint32_t *>(out);
        x0 += __uint_as_float(o << 16), x1 += __uint_as_float(o & 0xFFFF0000u);
    }
    if (g.bias != nullptr) x0 += b0, x1 += b1;
    union {
        bf16x2_t h;
        uint32_t u;
    } o;
    o.h = __builtin_convertvector((f32x2_t){x0, x1}, bf16x2_t);  // nearest even
    *reinterpret_cast<uint32_t *>(out) = o.u;
}

template <int AMODE, int BMODE, bool SINGLE>
__global__ void __launch_bounds__(kFewThreads) few_tile_kernel(GemmArgs g) {
    __shared__ __attribute__((aligned(16))) unsigned char lds[FewTile::LDS_BYTES];
    few_tile<AMODE, BMODE, SINGLE>(g, lds, blockIdx.x, gridDim.x);
}

// ---------------------------------------------------------------------------------------------
// Sketch products: S^T (generated by the work-group into LDS) times A [token][column], in a pipeline like that of
// gemm_tile: steps of 64 tokens, two stages, one barrier, A loaded straight into LDS, every instruction in its place.  A
// step of a 128 x 512 tile needs the matrix pipes for 2048 cycles, the vector units for 1700 (Gaussian entries: two chunks of
// eight per thread, a Philox call and four Box-Muller pairs each), and 64 KB from L2, which take about as long; they
// only fit beside each other if all three run all the time.  So the making of a step's entries is cut into units (a Philox
// round, half a Box-Muller pair) that are dealt evenly over the MFMAs between two barriers, from the last 16-deep step
// before one to the one in front of the next, and so are the loads over its first half.
// Rademacher: a thread's eight neighbours of one sketch column hold the calls of eight blocks of 128 tokens, one each
// (sixteen steps), and pass the words around.

// Eight Gaussian entries of one sketch column in the making.
struct GaussChunk {
    static constexpr int ROUNDS = 10, UNITS = ROUNDS + 8;
    uint32_t c0, c1, c2, c3;
    float rad;
    union {
        bf16x8_t v;
        bf16x2_t p[4];
    } out;
    __device__ __forceinline__ void unit(const SketchState &st, uint32_t block, uint32_t j, int u) {
        if (u == 0) c0 = block, c1 = j, c2 = st.off0, c3 = st.off1;
        if (u < ROUNDS) {
            philox_round(c0, c1, c2, c3, st.key0 + (uint32_t)u * kPhiloxBump0, st.key1 + (uint32_t)u * kPhiloxBump1);
            return;
        }
        const int q = (u - ROUNDS) / 2;
        const uint32_t w = q == 0 ? c0 : q == 1 ? c1 : q == 2 ? c2 : c3;
        if ((u - ROUNDS) % 2 == 0)
            rad = gauss_radius(w);
        else
            out.p[q] = gauss_pair(w, rad);
    }
};

template <typename S>
struct SketchTile {
    static constexpr int BM = S::BM, BN = S::BN, BK = S::BK, WM = S::WM, WN = S::WN, THREADS = S::THREADS;
    static constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    static constexpr int A_ELEMS = BM * BK, STAGE_ELEMS = (BM + BN) * BK, LDS_BYTES = 2 * STAGE_ELEMS * 2;
    static constexpr int GEN = BM * BK / 8 / THREADS;            // chunks of eight entries a thread generates per step
    static constexpr int LOADS = BN * BK * 2 / 1024 / (THREADS / 64);  // 1 KB loads per wave and step
    static_assert(BK == 64 && BM * BK / 8 % THREADS == 0 && BN * BK * 2 % (1024 * THREADS / 64) == 0, "shares of a thread");
    static_assert(BM % (32 * WM) == 0 && BN % (32 * WN) == 0 && BN % 128 == 0, "tile shape");
};

// Tile number `tile` of the product, tokens kk_begin .. kk_begin + kk - 1 (at least one).
template <typename S, int KIND>
__device__ __forceinline__ void sketch_tile(const GemmArgs &g, bf16_t *lds, int64_t tile, int64_t kk_begin, int kk, int slice) {
    typedef SketchTile<S> T;
    constexpr int BM = T::BM, BN = T::BN, BK = T::BK, TM = T::TM, TN = T::TN;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave / T::WN, wn = wave % T::WN;
    int64_t m0, n0;
    tile_origin<BM, BN>((uint32_t)tile, (uint32_t)((g.M + BM - 1) / BM), (uint32_t)((g.N + BN - 1) / BN), m0, n0);
    const int steps = (kk + BK - 1) / BK;
    const int stagger = (int)((uint32_t)tile / 8 % (uint32_t)steps);
    struct Tokens {  // of the slice: rows of A, and the first token of the step
        StepRows rows;
        u32x4_t ready;
        uint32_t step_token = 0;
        __device__ __forceinline__ void prepare(const Walk &w, bool last, bool live) {
            // (past the end it stays: the first tokens of the slice may be of another 1024, a generator call for nothing)
            ready = rows.descriptor(last, live), step_token = live ? w.soff / 2 : step_token;
        }
    } tokens;
    Walk walk;
    walk.init(kk, stagger), tokens.rows.init(g.B + kk_begin * g.ldb, g.ldb, kk, walk);

    constexpr uint32_t OOB = 0x80000000u;
    constexpr int CPR = BN / 8;  // chunks per row
    uint32_t b_off[T::LOADS];
#pragma unroll
    for (int j = 0; j < T::LOADS; ++j) {
        const int c = (wave * T::LOADS + j) * 64 + lane, row = c / CPR, col = col_chunk<BN>(row, c % CPR) * 8;
        b_off[j] = n0 + col < g.N ? (uint32_t)((row * g.ldb + n0 + col) * 2) : OOB;
    }
    typedef __attribute__((address_space(3))) bf16_t *lds_ptr_t;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr_t)lds;
    u32x4_t rsrc;  // of the step of A that is being requested
    uint32_t to;
    uint32_t making = 0;  // first token of the step whose entries are being made (tokens are below 2^31)
    auto begin_loads = [&](int stage) {  // (past the end: zeros, and the entries of a step that exists, not used)
        to = lds0 + (uint32_t)((stage * T::STAGE_ELEMS + T::A_ELEMS) * 2 + wave * T::LOADS * 1024);
        making = (uint32_t)kk_begin + tokens.step_token;
        rsrc = tokens.ready, settle(rsrc);
    };
    auto load = [&](int j) { load_to_lds(rsrc, to + j * 1024, b_off[j]); };

    // Chunk q of this thread: tokens gen_k * 8 .. + 7 of the step, sketch column m0 + gen_row + q * ROWS.  Tokens past the
    // slice are generated too: their rows of A are zeros.
    constexpr int ROWS = T::THREADS / (BK / 8);
    const int gen_row = tid / (BK / 8), gen_k = tid % (BK / 8);
    constexpr int UNITS = KIND == 0 ? GaussChunk::UNITS : 2;  // per chunk
    GaussChunk gauss;
    uint32_t words[KIND == 0 ? 1 : T::GEN][4] = {};  // Rademacher: of block 8 * held + gen_k
    uint32_t low = 0, high = 0;
    uint32_t held = 0xFFFFFFFFu;
    bf16_t *made = lds;
    auto begin_entries = [&](int stage) {
        made = lds + stage * T::STAGE_ELEMS;
        if constexpr (KIND != 0) {
            if ((making >> 10) != held) {
                held = making >> 10;
#pragma unroll
                for (int q = 0; q < T::GEN; ++q) {
                    const Words4 w = philox4x32_10(held * 8 + gen_k, (uint32_t)(m0 + gen_row + q * ROWS), g.st.off0,
                                                   g.st.off1, g.st.key0, g.st.key1);
#pragma unroll
                    for (int x = 0; x < 4; ++x) words[q][x] = w.w[x];
                }
            }
        }
    };
    auto unit = [&](int u) {
        const int q = u / UNITS, part = u % UNITS, row = gen_row + q * ROWS;
        bf16_t *dst = made + row * BK + kchunk_pos<BK>(row, gen_k) * 8;
        if constexpr (KIND == 0) {
            gauss.unit(g.st, (making >> 3) + gen_k, (uint32_t)(m0 + row), part);
            if (part == UNITS - 1) *reinterpret_cast<bf16x8_t *>(dst) = gauss.out.v;
        } else if (part == 0) {
            // the two words of the step's 64 tokens, from the neighbour that holds their block
            const int from = (lane & ~7) | (int)((making >> 7) & 7);
            const bool second = (making & 64) != 0;
            const uint32_t w0 = words[q][0], w1 = words[q][1], w2 = words[q][2], w3 = words[q][3];
            low = __shfl(second ? w2 : w0, from, 64);
            high = __shfl(second ? w3 : w1, from, 64);
        } else {
            *reinterpret_cast<bf16x8_t *>(dst) = radem_operand(((gen_k & 4) != 0 ? high : low) >> (8 * (gen_k & 3)));
        }
    };

    f32x16_t acc[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.0f;
    struct Frags {
        bf16x8_t a[TM], b[TN];
    };
    auto read = [&](Frags &f, int stage, int ks, int i) {  // fragment i of a 16-deep step
        const bf16_t *As = lds + stage * T::STAGE_ELEMS, *Bs = As + T::A_ELEMS;
        if (i < TN)
            f.b[i] = frag_columns<BN>(Bs, wn * (BN / T::WN) + i * 32, ks * 16, lane);
        else
            f.a[i - TN] = frag_kcontig<BK>(As, wm * (BM / T::WM) + (i - TN) * 32, ks * 16, lane);
    };
    constexpr int FRAGS = TM + TN, MFMAS = TM * TN, KS = BK / 16, SLOTS = KS * MFMAS, ALL = T::GEN * UNITS, HALF = (T::LOADS + 1) / 2;
    // One 16-deep step, number `place` of the four from barrier to barrier: multiplies `now`, reads the fragments of the one behind it.
    auto sixteen = [&](const Frags &now, Frags &next, int stage, int ks, int place) {
#pragma unroll
        for (int i = 0; i < MFMAS; ++i) {
            const int a = i / TN, b = i % TN, slot = place * MFMAS + i;
            acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(now.b[b], now.a[a], acc[a][b], 0, 0, 0);
#pragma unroll
            for (int r = i * FRAGS / MFMAS; r < (i + 1) * FRAGS / MFMAS; ++r) read(next, stage, ks, r);
            if (place < 2) {
#pragma unroll
                for (int r = i * HALF / MFMAS; r < (i + 1) * HALF / MFMAS; ++r)
                    if (place * HALF + r < T::LOADS) load(place * HALF + r);
            }
#pragma unroll
            for (int u = slot * ALL / SLOTS; u < (slot + 1) * ALL / SLOTS; ++u) unit(u);
            // (+-1: short steps, which wait for their loads; what the next ones need is made while they do)
            if (KIND != 0 ? place == KS - 1 && i == MFMAS - 1 : place == 1 && i == MFMAS / 2) prepare_step(walk, tokens);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // (the order of barrier, reads and loads: see gemm_tile)
    auto meet = [] {
        wait_for_loads<0>();
        __syncthreads();
    };
    Frags f[2];
    prepare_step(walk, tokens), begin_loads(0);
#pragma unroll
    for (int j = 0; j < T::LOADS; ++j) load(j);
    // The loads first.  (The compiler put the generator's first call in front of them, 55 instructions that wait for each other: +-1 products of
    // few steps were 1 % slower, 4096 x 768, k = 410 18.0 us instead of 17.8.)
    __builtin_amdgcn_sched_barrier(0);
    begin_entries(0);
#pragma unroll
    for (int u = 0; u < ALL; ++u) unit(u);
    meet();
#pragma unroll
    for (int i = 0; i < FRAGS; ++i) read(f[0], 0, 0, i);
    prepare_step(walk, tokens), begin_loads(1), begin_entries(1);
#pragma unroll
    for (int j = 0; j < HALF; ++j) load(j);
#pragma unroll
    for (int u = 0; u < MFMAS * ALL / SLOTS; ++u) unit(u);
    for (int t = 0; t < steps; ++t) {
        const int stage = t & 1;
#pragma unroll
        for (int ks = 0; ks < KS - 1; ++ks) sixteen(f[ks & 1], f[(ks + 1) & 1], stage, ks + 1, ks + 1);
        meet();
        begin_loads(stage), begin_entries(stage);
        sixteen(f[1], f[0], stage ^ 1, 0, 0);  // (past the end: what the stage holds, not used)
    }
    wait_for_loads<0>();
    __syncthreads();
    char *strip = reinterpret_cast<char *>(lds) + wave * kStripBytes;
    if (g.direct)
        write_tile<true, false, false, TM, TN, 1>(g, acc, strip, m0, n0, wm, wn, 0, lane, slice);
    else
        write_tile<false, false, false, TM, TN, 1>(g, acc, strip, m0, n0, wm, wn, 0, lane, slice);
}

// Share `work` of a sketch product: a slice of a tile, or (the last ones) the short last slices of per_tail tiles.
template <typename S, int KIND>
__device__ __forceinline__ void sketch_share(const GemmArgs &g, bf16_t *lds, int work, int tiles) {
    auto renumbered = [](int x, int count) {  // an XCD (x % 8) takes a contiguous run, as in gemm_tile
        const int per = count / 8, rem = count % 8, xcd = x % 8;
        return xcd * per + (xcd < rem ? xcd : rem) + x / 8;
    };
    int tile, end, slice;
    int64_t begin, len = g.k_chunk;
    if (work < g.slices * tiles) {
        slice = work / tiles, tile = renumbered(work % tiles, tiles), end = tile + 1;
        begin = slice * g.k_chunk;
    } else {
        const int groups = (tiles + g.per_tail - 1) / g.per_tail;
        slice = g.slices, tile = renumbered(work - g.slices * tiles, groups) * g.per_tail, end = min(tiles, tile + g.per_tail);
        begin = slice * g.k_chunk;
    }
    len = min(len, g.K - begin);
    for (;;) {
        sketch_tile<S, KIND>(g, lds, tile, begin, (int)len, slice);
        if (++tile >= end) break;
        __syncthreads();  // (LDS is used again)
    }
}

template <typename S, int KIND>
__global__ void __launch_bounds__(S::THREADS) sketch_kernel(GemmArgs g, int tiles) {
    __shared__ __attribute__((aligned(1024))) bf16_t lds[SketchTile<S>::LDS_BYTES / 2];
    sketch_share<S, KIND>(g, lds, blockIdx.x, tiles);
}

template <typename S, int AMODE, int BMODE, int OUT>
__global__ void __launch_bounds__(S::THREADS) gemm_mfma_kernel(GemmArgs g) {
    __shared__ __attribute__((aligned(1024))) bf16_t lds[S::LDS_BYTES / 2];
    gemm_tile<S, AMODE, BMODE, OUT>(g, lds, blockIdx.x, gridDim.x);
}

// Two independent products in one launch: `blocks_a` work-groups are the tiles of a plain product
// (Y = X W^T or dX = dY W, rounded to bf16), `sketch_blocks` others the (tile, token slice) pairs
// of the sketch product of the same pass (fp32 partial results).  Neither fills the chip on its
// own at RoBERTa-base sizes (192 and 56 .. 252 work-groups on 256 compute units); issued as one
// grid, the sketch work-groups take the compute units the plain product leaves idle and the ones
// it frees first.  A separate launch per product cannot do that: two kernels do not share a
// compute unit when each needs most of its LDS.  The host decides which of the two comes first
// in the grid (`sketch_first`).
// `colsum_blocks` further work-groups, if any, take the column blocks of `gc` (the bias gradient,
// column sums of dY: a backward pass whose last round leaves compute units idle runs them in this
// launch, next to the products that read the same dY).  Grid order: plain tiles, sketch
// work-groups, column blocks; with `sketch_first` (few, long sketch work-groups, or a plain
// product that fills the chip by itself) sketch work-groups, column blocks, plain tiles: the
// column blocks then start on the compute units the sketch product leaves free, ahead of the
// plain tiles, instead of competing with the last round of plain tiles for memory.
// ShapeCompact with 64 x 256 sketch tiles: either needs half of a compute unit's LDS and registers, so two work-groups
// share one, and what one waits for (first loads, first entries, the writing of its tile) the other fills.
template <typename SA, typename SB>
constexpr int pair_waves_per_simd() { return SA::LDS_BYTES <= 80 * 1024 && SketchTile<SB>::LDS_BYTES <= 80 * 1024 ? 4 : 1; }
template <typename SA, int BMODE_A, typename SB, int KIND>
__global__ void __launch_bounds__(SA::THREADS, (pair_waves_per_simd<SA, SB>())) gemm_pair_kernel(GemmArgs ga, GemmArgs gb, int blocks_a, int tiles_b,
                                                                 int sketch_blocks, int colsum_blocks, int sketch_first,
                                                                 ColsumArgs gc) {
    typedef SketchTile<SB> TB;
    static_assert(SA::THREADS == SB::THREADS, "both halves run with the same work-group size");
    constexpr int BYTES = SA::LDS_BYTES > TB::LDS_BYTES ? SA::LDS_BYTES : TB::LDS_BYTES;
    static_assert(BYTES >= kColsumLdsFloats * 4, "room for the column sums");
    __shared__ __attribute__((aligned(1024))) bf16_t lds[BYTES / 2];
    const int b = (int)blockIdx.x;
    const int a = sketch_first ? b - sketch_blocks - colsum_blocks : b;  // index among the plain tiles
    const int i = sketch_first ? b : b - blocks_a;                       // index among the sketch work-groups
    const int c = sketch_first ? b - sketch_blocks : b - blocks_a - sketch_blocks;  // index among the column blocks
    if (a >= 0 && a < blocks_a)
        gemm_tile<SA, A_KCONTIG, BMODE_A, OUT_BF16>(ga, lds, a, blocks_a);
    else if (i >= 0 && i < sketch_blocks)
        sketch_share<SB, KIND>(gb, lds, i, tiles_b);
    else
        colsum_body<bf16_t>(gc, reinterpret_cast<float *>(lds), c, colsum_blocks);
}

// dW = G^T X_proj and db = dY^T 1 in one launch: the first `blocks_a` work-groups are the tiles of
// dW, the others the column blocks of dY.  The two do not depend on each other; dW has few tiles
// and a short contraction (k), so its launch leaves compute units idle and is over in a few
// microseconds, most of them latency: the column sums, bound by memory, run beside it for free.
template <typename S>
__global__ void __launch_bounds__(S::THREADS) dw_colsum_kernel(GemmArgs g, ColsumArgs c, int blocks_a) {
    static_assert(S::LDS_BYTES >= kColsumLdsFloats * 4, "room for the column sums");
    __shared__ __attribute__((aligned(1024))) bf16_t lds[S::LDS_BYTES / 2];
    if ((int)blockIdx.x < blocks_a)
        gemm_tile<S, A_MCONTIG, B_NCONTIG, OUT_BF16>(g, lds, blockIdx.x, blocks_a);
    else
        colsum_body<bf16_t>(c, reinterpret_cast<float *>(lds), (int64_t)blockIdx.x - blocks_a, (int64_t)gridDim.x - blocks_a);
}

// |X^T dY|_F^2 per tile and the row norms of X and dY (variance monitors) in one launch: the product has
// few tiles and a long contraction, so the row norms, bound by memory, run on the compute units it leaves
// idle (or ahead of its last round) instead of in a pass of their own.
// (ShapeCompact: two work-groups to a compute unit)
template <typename S>
__global__ void __launch_bounds__(S::THREADS, S::SA == 2 ? 4 : 1) xty_norms_kernel(GemmArgs g, RowNormArgs r, int tiles) {
    __shared__ __attribute__((aligned(1024))) bf16_t lds[S::LDS_BYTES / 2];
    if ((int)blockIdx.x < tiles)
        gemm_tile<S, A_MCONTIG, B_NCONTIG, OUT_SUMSQ>(g, lds, blockIdx.x, tiles);
    else
        row_norms_body<bf16_t>(r, reinterpret_cast<double *>(lds), (int64_t)blockIdx.x - tiles, (int64_t)gridDim.x - tiles);
}

// dW and db where dW runs on few_tile.
template <bool SINGLE>
__global__ void __launch_bounds__(kFewThreads) few_dw_colsum_kernel(GemmArgs g, ColsumArgs c, int blocks_a) {
    constexpr int BYTES = FewTile::LDS_BYTES;
    static_assert(BYTES >= kColsumLdsFloats * 4, "room for the column sums");
    __shared__ __attribute__((aligned(16))) unsigned char lds[BYTES];
    if ((int)blockIdx.x < blocks_a)
        few_tile<A_MCONTIG, B_NCONTIG, SINGLE>(g, lds, blockIdx.x, blocks_a);
    else
        colsum_body<bf16_t>(c, reinterpret_cast<float *>(lds), (int64_t)blockIdx.x - blocks_a, (int64_t)gridDim.x - blocks_a);
}

// out[r][c] (bf16) = alpha * sum_s part[s][r][c], the slices added in slice order; 4 columns per
// thread.  The loads of up to eight slices are issued together (slices past the end are skipped
// by predicate, not by a loop exit), so a thread waits for memory once per eight slices.
__global__ void __launch_bounds__(256) reduce_partials_kernel(const float *__restrict__ part, bf16_t *__restrict__ out,
                                                              int64_t elems, int splits, int64_t split_stride,
                                                              float alpha) {
    const int64_t e = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (e >= elems) return;
    float4 s = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    for (int z = 0; z < splits; z += 8) {
        float4 p[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (z + u < splits) p[u] = *reinterpret_cast<const float4 *>(part + (int64_t)(z + u) * split_stride + e);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (z + u >= splits) break;
            if (z + u == 0)
                s = p[0];  // not 0 + p: a sum that is -0 stays -0
            else
                s.x += p[u].x, s.y += p[u].y, s.z += p[u].z, s.w += p[u].w;
        }
    }
    uint2 o;
    o.x = (uint32_t)f32_to_bf16(alpha * s.x) | ((uint32_t)f32_to_bf16(alpha * s.y) << 16);
    o.y = (uint32_t)f32_to_bf16(alpha * s.z) | ((uint32_t)f32_to_bf16(alpha * s.w) << 16);
    *reinterpret_cast<uint2 *>(out + e) = o;
}

// ---------------------------------------------------------------------------------------------
// Small sketch sizes (k <= 64): S^T A is bound by reading A once from HBM, so this kernel is a
// streaming pass.  A work-group owns BN columns and one slice of tokens and walks the slice 64
// tokens at a time.  The four waves split the contraction: wave w takes tokens 16w .. 16w+15 of
// every step, for all 32*TM sketch columns and all BN operand columns, so every sketch entry is
// generated exactly once per work-group and the generator's ALU work stays far below the memory
// time.  A wave loads exactly the 16 token rows it consumes (global -> registers, D steps in
// flight; measured: 2 is faster than 1, 3, 4 and 6 at every size), passes them through its own
// part of LDS (the MFMA wants 8 consecutive tokens of one column per lane, memory has 8
// consecutive columns of one token: the transposing LDS read turns one into the other) and never
// waits for another wave inside the loop.  At the end the four
// partial accumulators are summed through LDS and written as fp32 partials of the slice (or,
// with a single slice, scaled and rounded to bf16).
struct SmallkArgs {
    const bf16_t *A;  // n x d
    void *C;          // bf16 k x d, or fp32 partials [slice][k][d]
    int64_t n, d, k;
    int64_t k_chunk;  // tokens per slice (multiple of 128)
    float alpha;
    SketchState st;
};

template <int TM, int BN, int KIND, int D, int OUT>
__global__ void __launch_bounds__(256) sketch_smallk_kernel(SmallkArgs g) {
    static_assert(BN == 128 || BN == 256, "columns per work-group");
    constexpr int BK = 64, STRIDE = BN + TPAD, STAGE_ELEMS = BK * STRIDE, CHUNKS = BN * BK / 8 / 256;
    constexpr int TN = BN / 32;
    constexpr int PITCH = 128 * 4 + 16;  // bytes per row of a region of the final sum
    constexpr int LDS_BYTES = 2 * STAGE_ELEMS * 2 > 4 * 32 * PITCH ? 2 * STAGE_ELEMS * 2 : 4 * 32 * PITCH;
    __shared__ __attribute__((aligned(16))) bf16_t lds[LDS_BYTES / 2];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t n0 = (int64_t)blockIdx.x * BN;
    const int64_t kk_begin = (int64_t)blockIdx.y * g.k_chunk;
    const int kk_len = (int)(min(g.n, kk_begin + g.k_chunk) - kk_begin);  // >= 1: the host makes no empty slice
    const int num_tiles = (kk_len + BK - 1) / BK;

    // Byte offsets from the first token row of a step (2^31 = reads as zero: columns beyond d); the
    // buffer descriptor is re-based on that row at every step and covers the step's rows only, so
    // tokens beyond the slice read as zeros and A may have any size.
    constexpr uint32_t OOB = 0x80000000u;
    uint32_t off[CHUNKS];
    int lds_of[CHUNKS];
    constexpr int CPR = BN / 8, RPI = 64 / CPR;  // chunks per row; rows per load instruction of a wave
    static_assert(CHUNKS * RPI == 16, "a wave's loads of a step cover its 16 rows");
#pragma unroll
    for (int q = 0; q < CHUNKS; ++q) {  // wave w: rows 16w .. 16w+15 of the step, CPR consecutive lanes per row
        const int row = 16 * wave + RPI * q + lane / CPR, nc = lane % CPR;
        lds_of[q] = row * STRIDE + nc * 8;
        off[q] = n0 + nc * 8 < g.d ? (uint32_t)((row * g.d + n0 + nc * 8) * 2) : OOB;
    }

    u32x4_t rb[D][CHUNKS];
    auto issue = [&](int set, int t) {
        const int rows = min(BK, kk_len - t * BK);  // <= 0 for every t >= num_tiles
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<bf16_t *>(g.A + (kk_begin + (int64_t)t * BK) * g.d), (short)0,
            __builtin_amdgcn_readfirstlane((int)((rows > 0 ? rows : 0) * g.d * 2)), 0x00020000);
#pragma unroll
        for (int q = 0; q < CHUNKS; ++q)  // aux 2 = non-temporal: A is read once and should not displace anything
            rb[set][q] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, off[q], 0, 2);
    };
    auto store_lds = [&](int set, int stage) {
#pragma unroll
        for (int q = 0; q < CHUNKS; ++q)
            *reinterpret_cast<u32x4_t *>(lds + stage * STAGE_ELEMS + lds_of[q]) = rb[set][q];
    };

    f32x16_t acc[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.0f;

    // The rows a wave writes to LDS are the rows it reads back, so the order that matters is the
    // one between lanes of a wave (LDS serves a wave's instructions in order).
    auto wave_sync = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
#pragma unroll
    for (int s = 0; s < D; ++s) issue(s, s);
    store_lds(0, 0);
    wave_sync();
    const int groups = (num_tiles + D - 1) / D;
    for (int grp = 0; grp < groups; ++grp) {
#pragma unroll
        for (int s = 0; s < D; ++s) {
            const int t = grp * D + s;
            issue(s, t + D);
            if (t < num_tiles) {
                const bf16_t *Bs = lds + (t & 1) * STAGE_ELEMS;
                const int tok = (int)kk_begin + t * BK + 16 * wave + ((lane >> 5) << 3);  // this lane's first token
                bf16x8_t af[TM], bfr[TN];
#pragma unroll
                for (int a = 0; a < TM; ++a) {
                    const uint32_t j = (uint32_t)(a * 32 + (lane & 31));
                    if constexpr (KIND == 0) {
                        af[a] = gauss_operand(g.st, (uint32_t)(tok >> 3), j);
                    } else {
                        const Words4 rw =
                            philox4x32_10((uint32_t)(tok >> 7), j, g.st.off0, g.st.off1, g.st.key0, g.st.key1);
                        af[a] = radem_operand(rw, (uint32_t)tok);
                    }
                }
#pragma unroll
                for (int b = 0; b < TN; ++b) bfr[b] = frag_transposed(Bs, STRIDE, b * 32, 16 * wave, lane);
#pragma unroll
                for (int a = 0; a < TM; ++a)
#pragma unroll
                    for (int b = 0; b < TN; ++b)
                        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[b], af[a], acc[a][b], 0, 0, 0);
            }
            store_lds((s + 1) % D, (t + 1) & 1);
            wave_sync();  // this wave has consumed its rows of step t and sees its rows of step t+1
        }
    }
    __syncthreads();  // every wave is done with its rows: LDS is free for the sum below

    // Sum the four waves' accumulators, 32 rows x 128 columns at a time: every wave puts its block
    // into its own LDS region, then all threads add the four regions and write full rows.
    // (Accumulator register v of lane l is C(l % 32, 8*(v/4) + 4*(l/32) + v%4) of a 32x32 tile.)
    char *region = reinterpret_cast<char *>(lds);
    const int r = lane & 31, h = lane >> 5;
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int half = 0; half < BN / 128; ++half) {
#pragma unroll
            for (int bb = 0; bb < 4; ++bb)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x16_t &t = acc[a][half * 4 + bb];
                    *reinterpret_cast<float4 *>(region + (wave * 32 + r) * PITCH + (bb * 32 + 8 * q + 4 * h) * 4) =
                        make_float4(t[4 * q], t[4 * q + 1], t[4 * q + 2], t[4 * q + 3]);
                }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int f = tid + 256 * i, row = f >> 5, c4 = f & 31;
                float4 s = *reinterpret_cast<const float4 *>(region + row * PITCH + c4 * 16);
#pragma unroll
                for (int w = 1; w < 4; ++w) {
                    const float4 p = *reinterpret_cast<const float4 *>(region + (w * 32 + row) * PITCH + c4 * 16);
                    s.x += p.x, s.y += p.y, s.z += p.z, s.w += p.w;
                }
                const int64_t grow = a * 32 + row, gcol = n0 + half * 128 + c4 * 4;
                if (grow < g.k && gcol < g.d) {  // d is a multiple of 4
                    if constexpr (OUT == OUT_BF16) {
                        union {
                            bf16x2_t hh[2];
                            uint2 u;
                        } o;
                        o.hh[0] = __builtin_convertvector((f32x2_t){g.alpha * s.x, g.alpha * s.y}, bf16x2_t);
                        o.hh[1] = __builtin_convertvector((f32x2_t){g.alpha * s.z, g.alpha * s.w}, bf16x2_t);
                        *reinterpret_cast<uint2 *>(reinterpret_cast<bf16_t *>(g.C) + grow * g.d + gcol) = o.u;
                    } else {
                        *reinterpret_cast<float4 *>(reinterpret_cast<float *>(g.C) +
                                                    ((int64_t)blockIdx.y * g.k + grow) * g.d + gcol) = s;
                    }
                }
            }
            __syncthreads();
        }
}

}  // namespace

}  // namespace rmm
