// Tiled products for the fp32 data path of the layer, and for the bf16 shapes that the bf16 kernels
// (mfma_kernels.hpp) do not take:
//
//   C[M x N] = alpha * A B (+ bias) (+ old C),   A in memory either way round or P^T generated on
//   chip, B in memory either way round, accumulation in fp32.
//
// An fp32 number is the exact sum of three bf16 numbers (24 significant bits = 3 x 8: round to
// nearest, subtract, round, subtract; the last rest fits), so an fp32 product runs on the bf16 matrix
// pipes: the operand tiles are split on their way into LDS (three planes) and a 32x32x16 block is the
// sum of eight bf16 MFMAs, every pair of planes but the last with the last, whose share is below 2^-32
// of a product.  Each plane product is exact in fp32, so what rounds is the fp32 accumulation; with the
// products of the two first planes summed apart from the smaller ones its error is below that of a chain of fp32
// multiply-adds at every size looked at (a third of it at 4096 x 768 -> 3072 with normal entries; in one sum it was
// 12 % above it there with entries over 40 binades).  Operands that are bf16 already, and the +-1 entries of the Rademacher and
// SORS sketches, are one plane.
//
// The whole range of fp32 is served.  bf16 has fp32's exponents, so below 2^-110 the lower planes would lose
// bits: fp32 operands are multiplied by 2^24 before they are split (fp32's smallest number becomes 2^-125), and the
// sums by the inverse.  Operands from about 2^104 up, infinities and sums that leave fp32 with the factors on them
// then end as an infinity or NaN in the accumulator, NaN operands as NaN: the outputs where that happened are
// computed again with fp32 multiply-adds, element by element (plain_dot), and get what those give.  That is slow
// where it is many: 4096 x 768 -> 3072 forward, 0.21 ms; all of X NaN 0.23 (a NaN ends its sum at once), one row of X
// at the lowest fp32 value 3.6 (every sketch sum meets it), all of X around 1e34 21 ms.
//
// Why not v_mfma_f32_32x32x2_f32: it runs on the vector units' fp32 multipliers (measured on this
// chip: 72 cycles plus 4 for every vector instruction beside it), 576 cycles for the block that takes
// 8 x 32 here, and address arithmetic, splitting and the sketch generator would add to that instead of
// running beside it.
#pragma once
#include <type_traits>

#include "colsum.hpp"
#include "mfma_frag.hpp"
#include "tile_range.hpp"

namespace rmm {

enum { PA_K = 0, PA_M = 1, PA_GAUSS = 2, PA_SIGN = 3 };  // A[m][kk] / A[kk][m] / P^T(m, kk) generated: Gaussian / +-1 entries
enum { PB_K = 0, PB_N = 1 };                             // B[n][kk] / B[kk][n]

struct PlainArgs {
    const void *A;
    int64_t lda;
    const void *B;
    int64_t ldb;
    void *C;
    int64_t ldc;
    const void *bias;
    int64_t M, N, K;
    float alpha;
    int accumulate;
    int kind;  // sketch operand only
    SketchState st;
    // bf16 sketch products only: a tile's tokens in `slices` runs of k_chunk (a multiple of 128), a work-group each; with more
    // than one they write fp32 sums, unscaled, split_stride elements apart, which reduce_slices_kernel adds.
    int slices;
    int64_t k_chunk, split_stride;
};

namespace {

// BM x BN outputs, BK contraction elements per LDS tile, WM x WN waves over the tile, WK waves that
// take a share of each tile's contraction; always eight waves, two per SIMD, so that one wave's
// splitting, LDS traffic and generator work run beside the other's MFMAs.
constexpr int kPlainThreads = 512;
template <int BM_, int BN_, int BK_, int WM_, int WN_, int WK_>
struct PlainShape {
    static constexpr int BM = BM_, BN = BN_, BK = BK_, WM = WM_, WN = WN_, WK = WK_;
    static_assert(64 * WM * WN * WK == kPlainThreads, "eight waves");
};
typedef PlainShape<128, 128, 32, 2, 4, 1> PlainBig;    // most flops per byte
typedef PlainShape<64, 64, 64, 2, 2, 2> PlainMid;      // four times as many tiles
typedef PlainShape<32, 32, 128, 1, 1, 8> PlainTiny;    // few tiles: short chains, each wave an eighth of the contraction
typedef PlainShape<32, 128, 64, 1, 4, 2> PlainSketch;  // sketch products: an entry is generated once per 128 columns

// LDS by byte address: one register an operand, stage and 16-deep step, everything else in the offsets of the instructions.  (The
// compiler keeps an address for every fragment otherwise, some thirty, and spills sums for them: `opaque` keeps it from it.)
template <typename V>
__device__ __forceinline__ __attribute__((address_space(3))) V *lds_at(uint32_t byte) {
    return (__attribute__((address_space(3))) V *)(uintptr_t)byte;
}
__device__ __forceinline__ uint32_t lds_byte(void *p) {
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)p;
}
__device__ __forceinline__ uint32_t opaque(uint32_t x) {
    asm("" : "+v"(x));
    return x;
}

// How an operand is loaded: 4 = 16-byte buffer loads (every row on 16 bytes; bf16: a whole number of them); 3 = the same for
// rows that start anywhere; both with 32-bit offsets inside a tile (rows below 2^22 elements).
// 0 = element loads from 64-bit addresses, for longer rows.  Of bf16 operands in one product one may be 4 and the other 3.
template <typename T>
constexpr int plain_planes() { return sizeof(T) == 4 ? 3 : 1; }

template <typename T, typename S, int AMODE, int BMODE>
struct PlainTile {
    static constexpr bool A_KROWS = AMODE != PA_M, B_KROWS = BMODE == PB_K;  // LDS tile [row][contraction] or [contraction][row]
    static constexpr int PA = AMODE == PA_GAUSS ? 3 : AMODE == PA_SIGN ? 1 : plain_planes<T>(), PB = plain_planes<T>();
    // (rows of 64 or 192 bytes modulo 256 keep the transposing reads off each other's banks)
    static constexpr int SA = A_KROWS ? S::BK : S::BM % 64 == 0 ? S::BM + TPAD : S::BM;
    static constexpr int SB = B_KROWS ? S::BK : S::BN % 64 == 0 ? S::BN + TPAD : S::BN;
    static constexpr int A_PLANE = (A_KROWS ? S::BM : S::BK) * SA, B_PLANE = (B_KROWS ? S::BN : S::BK) * SB;
    static constexpr int STAGE = PA * A_PLANE + PB * B_PLANE;  // bf16 elements
    static constexpr int RED_BYTES = S::WK > 1 ? 8 * 16 * 64 * 4 : 0;  // cross-wave sum
    static constexpr int LDS_BYTES = 2 * STAGE * 2 > RED_BYTES ? 2 * STAGE * 2 : RED_BYTES;
};

// Eight fp32 values as three bf16 vectors whose sum they are, a pair at a time.  (An infinity, or a number that rounds to one
// in bf16: infinity, NaN, NaN.)
struct Planes {
    union {
        bf16x8_t v;
        bf16x2_t h[4];
        uint32_t w[4];
    } p[3];
    __device__ __forceinline__ void split(int q, float x, float y) {
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            p[s].h[q] = __builtin_convertvector((f32x2_t){x, y}, bf16x2_t);  // nearest even
            if (s < 2) {
                x -= __uint_as_float(p[s].w[q] << 16);
                y -= __uint_as_float(p[s].w[q] & 0xFFFF0000u);
            }
        }
    }
};
// The pairs of planes that a product of operands of PA and PB planes is made of, smallest products first.
template <int PA, int PB>
struct PlaneProducts {
    int a[9] = {}, b[9] = {};
    static constexpr int COUNT = PA * PB - (PA + PB == 6);
    constexpr PlaneProducts() {
        int i = 0;
        for (int order = PA + PB - 2; order >= 0; --order)
            for (int s = 0; s < PA; ++s)
                if (order - s >= 0 && order - s < PB && order <= 3) a[i] = s, b[i] = order - s, ++i;
    }
};
// The fragments of a step in the order in which its products leave them: those that are done with first can be
// overwritten by the next step's first.
template <int PA, int PB, int TM, int TN>
struct FragmentOrder {
    bool of_a[PA * TM + PB * TN] = {};
    int plane[PA * TM + PB * TN] = {}, tile[PA * TM + PB * TN] = {};
    constexpr FragmentOrder() {
        int i = 0;
        for (int p = PA > PB ? PA - 1 : PB - 1; p >= 0; --p) {
            for (int u = 0; p < PB && u < TN; ++u) plane[i] = p, tile[i] = u, ++i;
            for (int u = 0; p < PA && u < TM; ++u) of_a[i] = true, plane[i] = p, tile[i] = u, ++i;
        }
    }
};
constexpr float kSplitUp = 0x1p24f, kSplitDown = 0x1p-24f;

// One operand tile (ROWS rows or columns of the product x BK contraction elements) on its way from
// memory to LDS, in chunks of eight elements that are neighbours in memory.  KROWS: the chunk runs
// along the contraction.  Elements beyond the contraction become zeros; rows beyond the operand hold
// anything: they only reach outputs that are not stored.
//
// Modes 4 and 3: the buffer descriptor starts at the tile and moves along the contraction with scalar
// arithmetic; it ends with the dword that holds the last valid element, and every dword beyond it reads
// as zero, so an edge costs at most a compare and a select per load.  Mode 3 loads whole dwords too: a
// bf16 row that starts in the middle of one is shifted into place (a fifth dword and a funnel shift per
// chunk), and what a chunk holds beyond the end of its row is cleared in store().
template <typename T, int ROWS, int BK, bool KROWS, int MODE, int STRIDE, int PLANE>
struct PlainLoader {
    static constexpr int CHUNKS = ROWS * BK / 8 / kPlainThreads, ES = (int)sizeof(T);
    static constexpr int WORDS = MODE == 0 ? 8 : ES == 4 ? 8 : MODE == 4 ? 4 : 5;  // registers of a chunk in flight
    static_assert(ROWS * BK % (8 * kPlainThreads) == 0, "whole chunks per thread");
    struct Regs {
        uint32_t v[CHUNKS][WORDS];
    };
    int kk[CHUNKS];
    uint32_t to[2][CHUNKS];  // of each LDS stage
    uint32_t off[CHUNKS];
    const T *p[MODE == 0 ? CHUNKS : 1];
    const T *base;
    int64_t ld;
    int rows_left;  // (dimensions are below 2^31)
    uint32_t skew = 0;  // bytes between the base and the first element
    int clamp[MODE == 0 ? CHUNKS : 1];

    __device__ __forceinline__ void init(const T *operand, int64_t ld_, int64_t row0, int64_t rows, int tid, uint32_t lds, uint32_t stage_bytes) {
        ld = ld_, rows_left = (int)(rows - row0);
        base = operand + (MODE == 0 ? 0 : row0 * (KROWS ? ld : 1));
        if constexpr (ES == 2 && MODE == 3) {  // descriptors start on a dword
            skew = (uint32_t)(reinterpret_cast<uintptr_t>(base) & 2u);
            base -= skew / 2;
        }
#pragma unroll
        for (int q = 0; q < CHUNKS; ++q) {
            const int c = tid + kPlainThreads * q;
            const int r = KROWS ? c / (BK / 8) : c % (ROWS / 8) * 8, k = KROWS ? c % (BK / 8) * 8 : c / (ROWS / 8);
            kk[q] = k;
            const uint32_t at = 2 * (KROWS ? r * STRIDE + kchunk_pos<BK>(r, k / 8) * 8 : k * STRIDE + r);
            to[0][q] = opaque(lds + at), to[1][q] = opaque(lds + stage_bytes + at);
            if constexpr (MODE == 0) {
                p[q] = operand + (KROWS ? min(row0 + r, rows - 1) * ld + k : k * ld + min(row0 + r, rows - 1));
                clamp[q] = KROWS ? 7 : (int)max((int64_t)0, min((int64_t)7, rows - 1 - row0 - r));  // last element of the chunk that exists
            } else {
                const uint32_t w = (uint32_t)ld;
                off[q] = r < rows_left ? (KROWS ? (uint32_t)r * w + (uint32_t)k : (uint32_t)k * w + (uint32_t)r) * ES + skew : 0x80000000u;
            }
        }
    }
    // Requests the next tile; `left` = contraction elements that remain (may be <= 0).
    __device__ __forceinline__ void load(Regs &g, int left) {
        if constexpr (MODE == 0) {
#pragma unroll
            for (int q = 0; q < CHUNKS; ++q) {
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const bool ok = kk[q] + (KROWS ? u : 0) < left;
                    const T *a = ok ? p[q] + min(u, clamp[q]) : base;  // an address that exists
                    g.v[q][u] = ES == 4 ? *reinterpret_cast<const uint32_t *>(a) : *reinterpret_cast<const uint16_t *>(a);
                }
                p[q] += KROWS ? BK : BK * ld;
            }
        } else {
            const int l = max(0, min(left, BK));
            const uint32_t bytes = tile_range_bytes<ES, KROWS, uint32_t>((uint32_t)rows_left, ROWS, (uint32_t)ld, (uint32_t)l, skew / ES);
            const __amdgpu_buffer_rsrc_t rsrc =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<T *>(base), (short)0,
                                                  __builtin_amdgcn_readfirstlane((int)min(bytes, 0x7FFFFFFCu)), 0x00020000);
#pragma unroll
            for (int q = 0; q < CHUNKS; ++q) {
#pragma unroll
                for (int h = 0; h < ES / 2; ++h) {
                    const bool ok = !KROWS || kk[q] + 4 * h < l;
                    const u32x4_t w = __builtin_amdgcn_raw_buffer_load_b128(rsrc, ok ? (off[q] & ~3u) + 16 * h : 0x80000000u, 0, 0);
#pragma unroll
                    for (int u = 0; u < 4; ++u) g.v[q][4 * h + u] = w[u];
                }
                if constexpr (ES == 2 && MODE == 3)
                    g.v[q][4] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, !KROWS || kk[q] < l ? (off[q] & ~3u) + 16 : 0x80000000u, 0, 0);
            }
            base += KROWS ? BK : BK * ld;
        }
    }
    // The way of a request's elements into LDS, in UNITS pieces that the caller deals between its MFMAs (fp32: a pair of elements
    // split, or the chunk's planes written).
    static constexpr int UNITS = CHUNKS * (ES == 4 ? 5 : 1);
    Planes planes;
    __device__ __forceinline__ void store(int unit, const Regs &g, int set, int left) {
        const int q = unit / (UNITS / CHUNKS), u = unit % (UNITS / CHUNKS);
        // (a select at the load would make every request wait for its data)
        const int valid = KROWS ? left - kk[q] : kk[q] < left ? 8 : 0;
        if constexpr (ES == 4) {
            if (u == 4) {
#pragma unroll
                for (int s = 0; s < 3; ++s) *lds_at<bf16x8_t>(to[set][q] + s * PLANE * 2) = planes.p[s].v;
                return;
            }
            float x = __uint_as_float(g.v[q][2 * u]), y = __uint_as_float(g.v[q][2 * u + 1]);
            if constexpr (MODE == 0 || (MODE == 3 && KROWS)) x = 2 * u < valid ? x : 0.0f, y = 2 * u + 1 < valid ? y : 0.0f;
            planes.split(u, x * kSplitUp, y * kSplitUp);
        } else if constexpr (MODE == 4) {  // (chunks lie wholly inside the operand or read as zeros)
            *lds_at<u32x4_t>(to[set][q]) = (u32x4_t){g.v[q][0], g.v[q][1], g.v[q][2], g.v[q][3]};
        } else {
            uint32_t w[4];
            if constexpr (MODE == 0) {
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] = g.v[q][2 * e] | g.v[q][2 * e + 1] << 16;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] = __builtin_amdgcn_alignbit(g.v[q][e + 1], g.v[q][e], (off[q] & 2u) * 8);
            }
            if constexpr (KROWS || MODE == 0) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    w[e] = 2 * e + 1 < valid ? w[e] : 2 * e < valid ? w[e] & 0xFFFFu : 0u;
            } else {  // (the descriptor's last dword may hold the first element behind the last row)
                w[0] = valid != 0 ? w[0] : 0u;
            }
            *lds_at<u32x4_t>(to[set][q]) = (u32x4_t){w[0], w[1], w[2], w[3]};
        }
    }
};

// Eight unscaled Gaussian entries P[t0 .. t0+7][j], t0 a multiple of 8.
__device__ __forceinline__ void gauss_eight_precise(const SketchState &st, uint32_t t0, uint32_t j, float (&v)[8]) {
    const Words4 r = philox4x32_10(t0 >> 3, j, st.off0, st.off1, st.key0, st.key1);
#pragma unroll
    for (int q = 0; q < 4; ++q) gauss_pair_precise(r.w[q], v[2 * q], v[2 * q + 1]);
}

// The same for the kinds whose entries are +1 and -1 (1 = Rademacher, 2 = SORS), as bf16.
__device__ __forceinline__ bf16x8_t sign_eight(int kind, const SketchState &st, uint32_t t0, uint32_t j) {
    const uint32_t t = t0 & 127u;
    const Words4 s = philox4x32_10(t0 >> 7, kind == 1 ? j : kSorsSignColumn, st.off0, st.off1, st.key0, st.key1);
    const uint32_t word = (t >> 5) == 0 ? s.w[0] : (t >> 5) == 1 ? s.w[1] : (t >> 5) == 2 ? s.w[2] : s.w[3];
    uint32_t bits = word >> (t & 31u);
    if (kind == 2) {
        const Words4 w = philox4x32_10(j >> 2, kSorsRowColumn, st.off0, st.off1, st.key0, st.key1);
        const uint32_t row = ((j & 3u) == 0 ? w.w[0] : (j & 3u) == 1 ? w.w[1] : (j & 3u) == 2 ? w.w[2] : w.w[3]) & st.row_mask;
#pragma unroll
        for (int u = 0; u < 8; ++u) bits ^= ((uint32_t)__popc(row & (t0 + u)) & 1u) << u;
    }
    union {
        bf16x8_t v;
        uint32_t d[4];
    } out;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        out.d[q] = 0x3F803F80u | (((bits >> (2 * q)) & 1u) << 15) | (((bits >> (2 * q + 1)) & 1u) << 31);
    return out.v;
}

// One output (of the contraction's elements k_begin .. k_end) by fp32 multiply-adds, unscaled; ends early where nothing can change the result any more.  A
// generated operand is made eight entries at a time (one generator call, eight loads of B in flight).
template <typename T, int AMODE, int BMODE>
__device__ __forceinline__ float plain_dot(const PlainArgs &g, int64_t r, int64_t c, int64_t k_begin, int64_t k_end) {
    constexpr bool GEN = AMODE == PA_GAUSS || AMODE == PA_SIGN;
    constexpr int STEP = GEN ? 8 : 1;
    const T *A = reinterpret_cast<const T *>(g.A), *B = reinterpret_cast<const T *>(g.B);
    float sum = 0.0f;
#pragma unroll 1
    for (int64_t k0 = k_begin; k0 < k_end && sum == sum; k0 += STEP) {
        float a[STEP];
        if constexpr (AMODE == PA_GAUSS) {
            gauss_eight_precise(g.st, (uint32_t)k0, (uint32_t)r, a);
        } else if constexpr (AMODE == PA_SIGN) {
            const bf16x8_t s = sign_eight(g.kind, g.st, (uint32_t)k0, (uint32_t)r);
#pragma unroll
            for (int u = 0; u < 8; ++u) a[u] = (float)s[u];
        } else {
            a[0] = load_f32<T>(AMODE == PA_K ? A + r * g.lda + k0 : A + k0 * g.lda + r);
        }
        float b[STEP];
#pragma unroll
        for (int u = 0; u < STEP; ++u)  // (entries beyond the contraction meet zeros)
            b[u] = !GEN || k0 + u < k_end ? load_f32<T>(BMODE == PB_K ? B + c * g.ldb + k0 + u : B + (k0 + u) * g.ldb + c) : 0.0f;
#pragma unroll
        for (int u = 0; u < STEP; ++u) sum = fmaf(a[u], b[u], sum);
    }
    return sum;
}

// Output tile number `block` of `blocks`.
template <typename T, typename Tout, typename S, int AMODE, int BMODE, int MODE_A, int MODE_B>
__device__ __forceinline__ void plain_tile(const PlainArgs &g, bf16_t *lds, int64_t block, int64_t blocks) {
    typedef PlainTile<T, S, AMODE, BMODE> L;
    constexpr int BM = S::BM, BN = S::BN, BK = S::BK, PA = L::PA, PB = L::PB;
    constexpr int TM = BM / S::WM / 32, TN = BN / S::WN / 32;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int kg = wave / (S::WM * S::WN), wm = wave % (S::WM * S::WN) / S::WN, wn = wave % S::WN;
    // Work-groups are dealt round-robin to the 8 XCDs: give each a contiguous run of positions, walked
    // in bands of 8 tile rows, so that work-groups that run together on one XCD share operands in its L2.
    // (32 bits: a grid has fewer than 2^31 work-groups, and a division of 64 bits is a microsecond in front of the first load)
    const uint32_t tiles_m = (uint32_t)((g.M + BM - 1) / BM), tiles_n = (uint32_t)((g.N + BN - 1) / BN);
    uint32_t tile;
    {
        const uint32_t per = (uint32_t)blocks / 8, rem = (uint32_t)blocks % 8, x = (uint32_t)block % 8, r = (uint32_t)block / 8;
        tile = x * per + (x < rem ? x : rem) + r;
    }
    constexpr bool GEN = AMODE == PA_GAUSS || AMODE == PA_SIGN, SLICED = GEN && sizeof(T) == 2;
    int64_t slice = 0, k_begin = 0, k_end = g.K;
    if constexpr (SLICED) {
        if (g.slices > 1) {  // (neighbours in a run of positions share their slice's rows of B)
            const uint32_t s = __builtin_amdgcn_readfirstlane(tile / (tiles_m * tiles_n));
            tile -= s * (tiles_m * tiles_n);
            slice = s, k_begin = s * g.k_chunk, k_end = min(k_end, k_begin + g.k_chunk);
        }
    }
    const int64_t len = k_end - k_begin;
    const uint32_t band = tile / (8 * tiles_n), in_band = tile - band * (8 * tiles_n);
    const uint32_t band_rows = min(8u, tiles_m - band * 8), in_col = in_band / band_rows;
    const int64_t m0 = (int64_t)(band * 8 + in_band - in_col * band_rows) * BM, n0 = (int64_t)in_col * BN;

    // With planes, the products of the two first planes are summed apart from the others, which are 2^-8 of them, and where a
    // wave has the whole contraction of a row-indexed operand (dX, dW) those of every other 16 elements in a sum of their
    // own: a large sum is then rounded once per 32 contraction elements instead of sixteen times, as it is on tiles whose
    // contraction two waves share.  (Y has always taken these tiles with one sum; a second one costs it 8 %.)
    constexpr bool PLANES = PA + PB > 2;
    constexpr int SUMS = PLANES && S::WK == 1 && BMODE == PB_N ? 2 : 1;
    f32x16_t acc[SUMS][TM][TN], low[PLANES ? TM : 1][PLANES ? TN : 1];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
#pragma unroll
                for (int x = 0; x < SUMS; ++x) acc[x][a][b][v] = 0.0f;
                if constexpr (PLANES) low[a][b][v] = 0.0f;
            }

    typedef PlainLoader<T, BN, BK, BMODE == PB_K, MODE_B, L::SB, L::B_PLANE> LoadB;
    typedef std::conditional_t<GEN, LoadB, PlainLoader<T, GEN ? BN : BM, BK, AMODE == PA_K, MODE_A, L::SA, L::A_PLANE>> LoadA;
    [[maybe_unused]] LoadA la;  // (not used by a generated operand)
    LoadB lb;
    const uint32_t lds0 = lds_byte(lds);
    constexpr uint32_t STAGE_BYTES = L::STAGE * 2;
    typename LoadA::Regs va[2];
    typename LoadB::Regs vb[2];
    if constexpr (!GEN) la.init(reinterpret_cast<const T *>(g.A), g.lda, m0, g.M, tid, lds0, STAGE_BYTES);
    lb.init(reinterpret_cast<const T *>(g.B) + (SLICED ? k_begin * g.ldb : 0), g.ldb, n0, g.N, tid, lds0 + PA * L::A_PLANE * 2, STAGE_BYTES);

    // (32 bits, as the tiles' ranges: uniform comparisons and products of 64 take vector instructions, some 30 in the way of every request
    // and every split.  Steps of fp32 and odd-width layers are 1 to 8 % shorter: 3000 x 768 -> 1001
    // bf16, k = 300, 64.3 -> 61.3 us, 569 x 538 -> 985 fp32, k = 57, 51.9 -> 49.1; 20 random fp32 steps 5.3 %.)
    uint32_t asked = 0;  // contraction elements requested so far
    auto left_of = [&](uint32_t from) { return (int)((uint32_t)len - from); };  // (dimensions are below 2^31)
    auto issue = [&](int set) {
        if constexpr (!GEN) la.load(va[set], left_of(asked));
        lb.load(vb[set], left_of(asked));
        asked += BK;
    };
    constexpr int STEPS = BK / 16 / S::WK;  // 16-deep contraction steps per tile and wave
    constexpr bool DEFER = STEPS > 1;  // a tile's last step is multiplied behind the next barrier
    // Tile t (in register set `set`) goes into LDS stage `set` in units: those of the loaders; the request of tile t + 2 into the same
    // registers; and those of a generated tile, which is made here, one chunk of eight tokens of a sketch column per thread, the waves
    // taking turns where the tile has fewer chunks than the work-group threads.  Entries beyond the operand meet zeros of B or are not
    // stored.  A chunk is one unit where a step is few MFMAs: cut up between these its instructions wait for each other.  It is the first
    // where tiles have several steps (3318 x 1145, k = 663 alone, bf16 50.3 us in pieces, 43.5 in one; +-1 entries, there behind the rest,
    // 29.3 and 26.9, fp32 51.3 and 46.6) and the last on tiles of one, which ask for the tile after next first (1000 x 512 -> 513, k = 100
    // bf16 forward 0.992 of the time).
    // PIECES: last and in units of half of the Philox rounds, or a pair of entries.  AHEAD: a chunk is begun one tile before the one that its
    // wave has to finish it for, so that all waves generate all the time (4096 x 3072, k = 410 fp32 alone 206 -> 197 us).
    constexpr int CALLS = BM * BK / 8, TURNS = GEN ? kPlainThreads / CALLS : 1;
    static_assert(!GEN || (CALLS % 64 == 0 && TURNS * CALLS == kPlainThreads && TURNS <= 2), "whole waves take turns, by the stage");
    constexpr bool PIECES = AMODE == PA_GAUSS && PB == 3, AHEAD = PIECES && TURNS == 2;
    constexpr int GEN_UNITS = PIECES ? (AHEAD ? 3 : 6) : GEN ? 1 : 0, A_UNITS = GEN ? 0 : LoadA::UNITS, B_UNITS = LoadB::UNITS,
                  UNITS = B_UNITS + A_UNITS + 1 + GEN_UNITS;
    const int gen_j = tid % CALLS / (BK / 8), gen_k = tid % CALLS % (BK / 8);
    uint32_t gen_to[2] = {};
    if constexpr (GEN) {
#pragma unroll
        for (int s = 0; s < 2; ++s) gen_to[s] = opaque(lds0 + s * STAGE_BYTES + 2 * (gen_j * L::SA + kchunk_pos<BK>(gen_j, gen_k) * 8));
    }
    const uint32_t column = (uint32_t)m0 + gen_j;
    auto token = [&](uint32_t t) { return (uint32_t)k_begin + t * BK + gen_k * 8; };
    auto turn = [&] {  // (opaque: two copies of everything else would move the sums from one to the other)
        int x = __builtin_amdgcn_readfirstlane(tid / CALLS);
        asm("" : "+s"(x));
        return x;
    };
    Words4 words{};
    [[maybe_unused]] Planes made;
    auto generate = [&](int part, int set, uint32_t t) __attribute__((always_inline)) {  // part 0 .. 5 of a Gaussian chunk
        uint32_t(&c)[4] = words.w;
        if (part == 0) c[0] = token(t) >> 3, c[1] = column, c[2] = g.st.off0, c[3] = g.st.off1;
        if (part < 2) {
#pragma unroll
            for (int r = 5 * part; r < 5 * part + 5; ++r)
                philox_round(c[0], c[1], c[2], c[3], g.st.key0 + (uint32_t)r * kPhiloxBump0, g.st.key1 + (uint32_t)r * kPhiloxBump1);
            return;
        }
        float x, y;
        gauss_pair_precise(c[part - 2], x, y);
        made.split(part - 2, x, y);
        if (part == 5) {
#pragma unroll
            for (int s = 0; s < PA; ++s) *lds_at<bf16x8_t>(gen_to[set] + s * L::A_PLANE * 2) = made.p[s].v;
        }
    };
    constexpr int CHUNK = DEFER ? 0 : UNITS - 1;
    auto put = [&](int unit, int set, uint32_t t) __attribute__((always_inline)) {
        if constexpr (GEN && !PIECES) {
            if (unit == CHUNK) {
                if (TURNS == 2 && turn() != set) return;
                if constexpr (AMODE == PA_SIGN) {
                    *lds_at<bf16x8_t>(gen_to[set]) = sign_eight(g.kind, g.st, token(t), column);
                } else {
#pragma unroll
                    for (int part = 0; part < 6; ++part) generate(part, set, t);
                }
                return;
            }
            unit -= CHUNK == 0;
        }
        if (unit < B_UNITS) return lb.store(unit, vb[set], set, left_of(t * BK));
        unit -= B_UNITS;
        if constexpr (!GEN) {
            if (unit < A_UNITS) return la.store(unit, va[set], set, left_of(t * BK));
        }
        unit -= A_UNITS;
        if (unit == 0) return issue(set);
        unit -= 1;
        if constexpr (PIECES) {
            if (!AHEAD) {
                generate(unit, set, t);
            } else if (turn() == set) {
                generate(unit + 3, set, t);
            } else {
                generate(unit, set ^ 1, t + 1);
            }
        }
    };
    struct Frags {
        bf16x8_t a[PA][TM], b[PB][TN];
    };
    static_assert(STEPS == 1 || STEPS % 2 == 0, "a tile's last step is in f[1]");
    Frags f[2];
    constexpr int FRAGS = PA * TM + PB * TN;
    constexpr FragmentOrder<PA, PB, TM, TN> order{};
    // (32 rows further down the chunks of a K-contiguous tile lie in the same places)
    uint32_t a_at[2][L::A_KROWS ? STEPS : 1], b_at[2][L::B_KROWS ? STEPS : 1];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int step = 0; step < STEPS; ++step) {
            const int k0 = (kg * STEPS + step) * 16, r0 = wm * (BM / S::WM), c0 = wn * (BN / S::WN);
            const uint32_t as = lds0 + s * STAGE_BYTES, bs = as + PA * L::A_PLANE * 2;
            if (L::A_KROWS || step == 0)
                a_at[s][step] = opaque(as + 2 * (L::A_KROWS ? kcontig_offset<BK>(r0, k0, lane) : transposed_offset(L::SA, r0, k0, lane)));
            if (L::B_KROWS || step == 0)
                b_at[s][step] = opaque(bs + 2 * (L::B_KROWS ? kcontig_offset<BK>(c0, k0, lane) : transposed_offset(L::SB, c0, k0, lane)));
        }
    auto columns = [](uint32_t at, int stride) { return frag_transposed(lds_at<s16x4_t>(at), lds_at<s16x4_t>(at + 8 * stride)); };
    auto fetch = [&](int i, Frags &to, int set, int step) __attribute__((always_inline)) {  // fragment i of a step
        const int p = order.plane[i], u = order.tile[i];
        if (order.of_a[i])
            to.a[p][u] = L::A_KROWS ? *lds_at<bf16x8_t>(a_at[set][L::A_KROWS ? step : 0] + 2 * (p * L::A_PLANE + u * 32 * L::SA))
                                    : columns(a_at[set][0] + 2 * (p * L::A_PLANE + step * 16 * L::SA + u * 32), L::SA);
        else
            to.b[p][u] = L::B_KROWS ? *lds_at<bf16x8_t>(b_at[set][L::B_KROWS ? step : 0] + 2 * (p * L::B_PLANE + u * 32 * L::SB))
                                    : columns(b_at[set][0] + 2 * (p * L::B_PLANE + step * 16 * L::SB + u * 32), L::SB);
    };
    constexpr PlaneProducts<PA, PB> products{};
    constexpr int MFMAS = PlaneProducts<PA, PB>::COUNT * TM * TN;  // of a step
    auto multiply = [&](int i, const Frags &x, int sum) __attribute__((always_inline)) {  // MFMA i of a step
        const int s = products.a[i / (TM * TN)], r = products.b[i / (TM * TN)], u = i % (TM * TN) / TN, w = i % TN;
        f32x16_t &to = s + r > 0 ? low[PLANES ? u : 0][PLANES ? w : 0] : acc[SUMS == 2 ? sum : 0][u][w];
        to = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x.a[s][u], x.b[r][w], to, 0, 0, 0);
    };

    // Two LDS stages, two register sets.  Between two barriers tile t is multiplied, t + 1 goes into LDS and t + 3 is requested (past
    // the end: zeros).  DEFER: a tile's barrier stands in front of the last step of the tile before it.  By then every wave holds
    // that step's fragments, so the stage can be written again, and the first fragments of the new tile are read under the last
    // step's MFMAs.  Where a product is eight MFMAs everything else is dealt between them (sched_barrier); in one piece it stands
    // behind the barrier for all waves at once.  With one step to a tile the fragments are read behind the barrier anyway, and the compiler
    // does better (fp32 400 x 3000 -> 500 forward 31.5 and 29.5 us, 834 x 2554 -> 1144 94.7 and 87.1) except beside generated entries of
    // fp32 sketches (2416 x 425 -> 192, k = 242 backward 1.026 and 1.004 of the time of code that fetches behind the barrier).
    // Against fetching behind the barrier, same bits: bf16 3000 x 768 -> 1001, k = 300, 61 -> 56 us a step, 209 x 424 -> 351 15.8 -> 13.4,
    // 830 x 472 -> 1269 +-1 35.3 -> 30.4; fp32 4096 x 768 -> 3072 dX and G 284 -> 262, 1906 x 69 -> 135, k = 191, 47.6 -> 44.9.
    // (What is left of the fp32 tiles' time is issue: a wave of the sketch tile has an instruction in flight 47 % of the time, and there
    // are two to a SIMD.)
    // FUNNEL: what shifts a request into place may not go in front of the barrier before its own: with both sets of the loop shifted at its
    // top, as the compiler has it, the newer request is waited for as well, right behind its issue (bf16 2132 x 2623 -> 1454 Y 68 us and 54,
    // 3000 x 1001 -> 768 28.2 and 23.0, 72 x 2461 -> 131, one step to a tile, 12.5 and 11.0).
    constexpr bool FUNNEL = sizeof(T) == 2 && !GEN && (MODE_A == 3 || MODE_B == 3);
    constexpr bool HOLD = DEFER ? PA + PB == 6 || FUNNEL : GEN && PLANES;
    constexpr int MAY_PASS = 0x8C;  // (scalar arithmetic, MFMAs and LDS)
    // COLUMNS: the same with one step to a tile, fp32 and both operands row-indexed (dW, monitors), where the first splits went in front of the
    // barrier and all waves waited there for a load: monitors of 8000 x 128 x 128 70 us and 65, 3338 x 201 x 167 41.2 and 38.1.
    constexpr bool COLUMNS = PLANES && !DEFER && AMODE == PA_M;
    const uint32_t num = ((uint32_t)len + BK - 1) / BK;
    // Short chains of fp32 tiles: those past the end are not split (256 x 128 -> 128: 18.6 -> 16 us a step).  Elsewhere the
    // branch costs more (Y 4096 x 768 -> 3072: 162 -> 175 us).
    constexpr bool SKIP = PB == 3 && S::WK == 8;
    // A step's fragments are read under the MFMAs READ_FROM to READ_TO of the step before.
    constexpr int READ_FROM = MFMAS >= 16 ? 4 : 0, READ_TO = MFMAS >= 16 ? MFMAS - 4 : MFMAS > 4 ? MFMAS - 2 : MFMAS;
    auto reads = [&](int i) { return i <= READ_FROM ? 0 : i >= READ_TO ? FRAGS : FRAGS * (i - READ_FROM) / (READ_TO - READ_FROM); };
    auto period = [&](auto first_, auto stage_, auto units_, uint32_t t) __attribute__((always_inline)) {
        constexpr bool FIRST = decltype(first_)::value;
        constexpr int s = decltype(stage_)::value, MAKE = decltype(units_)::value;
        constexpr int TOTAL = (FIRST && DEFER ? STEPS - 1 : STEPS) * MFMAS;
        constexpr int OVER = PLANES ? TOTAL - TOTAL / 8 : TOTAL;  // (the last ones done a while before the barrier)
        auto dealt = [](int x) { return x >= OVER ? MAKE : MAKE * x / OVER; };
        int m = 0;
        __syncthreads();
        if constexpr (FUNNEL && !DEFER) __builtin_amdgcn_sched_barrier(MAY_PASS);
        if constexpr (COLUMNS) __builtin_amdgcn_sched_barrier(0);
        if constexpr (FIRST || !DEFER) {
#pragma unroll
            for (int i = 0; i < FRAGS; ++i) fetch(i, f[0], s, 0);
        }
#pragma unroll
        for (int step = FIRST || !DEFER ? 0 : -1; step + DEFER < STEPS; ++step)
#pragma unroll
            for (int i = 0; i < MFMAS; ++i, ++m) {
                multiply(i, f[step & 1], step & 1);
                if constexpr (DEFER) {
#pragma unroll
                    for (int r = reads(i); r < reads(i + 1); ++r) fetch(r, f[(step + 1) & 1], s, step + 1);
                }
#pragma unroll
                for (int u = dealt(m); u < dealt(m + 1); ++u) put(u, s ^ 1, t + 1);
                if constexpr (HOLD) __builtin_amdgcn_sched_barrier(0);
            }
    };
    typedef std::integral_constant<int, 0> Stage0;
    typedef std::integral_constant<int, 1> Stage1;
    typedef std::integral_constant<int, UNITS> Everything;
    typedef std::integral_constant<int, 0> Nothing;
    issue(0);
    issue(1);
    if constexpr (AHEAD) {
#pragma unroll
        for (int part = 0; part < 3; ++part)
            if (turn() == 0) generate(part, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < UNITS; ++u) put(u, 0, 0);
    if (!SKIP || num > 1)
        period(std::true_type(), Stage0(), Everything(), 0);
    else
        period(std::true_type(), Stage0(), Nothing(), 0);
    uint32_t t = 1;
    for (; t + 1 < num; t += 2) {
        period(std::false_type(), Stage1(), Everything(), t);
        if (!SKIP || t + 2 < num)
            period(std::false_type(), Stage0(), Everything(), t + 1);
        else
            period(std::false_type(), Stage0(), Nothing(), t + 1);
    }
    if (t < num) period(std::false_type(), Stage1(), Nothing(), t);
    if constexpr (DEFER) {
#pragma unroll
        for (int i = 0; i < MFMAS; ++i) multiply(i, f[1], 1);
    }

    if constexpr (PLANES) {
#pragma unroll
        for (int u = 0; u < TM; ++u)
#pragma unroll
            for (int w = 0; w < TN; ++w) {
                if constexpr (SUMS == 2) acc[0][u][w] += acc[SUMS - 1][u][w];
                acc[0][u][w] += low[u][w];
            }
    }

    // Register v of lane l is C(8*(v/4) + 4*(l/32) + v%4, l % 32) of a 32x32 tile: a store instruction
    // writes two rows of 32 consecutive elements, whatever the alignment of the rows.
    Tout *C = reinterpret_cast<Tout *>(g.C);
    const T *bias = reinterpret_cast<const T *>(g.bias);
    const int half = lane >> 5;
    const float alpha = g.alpha * (PA == 3 && !GEN ? kSplitDown : 1.0f) * (PB == 3 ? kSplitDown : 1.0f);  // (exact)
    auto write = [&](int64_t r, int64_t c, float x, float scale, float bv) {
        if constexpr (SLICED) {
            if (g.slices > 1) {
                reinterpret_cast<float *>(g.C)[slice * g.split_stride + r * g.ldc + c] = x;
                return;
            }
        }
        x *= scale;
        if (g.bias != nullptr) x += bv;
        if (g.accumulate) x += load_f32<Tout>(C + r * g.ldc + c);
        store_f32<Tout>(C + r * g.ldc + c, x);
    };
    uint32_t open = 0;  // bit e: this lane's output number e is still to be made
    auto put_out = [&](int e, int64_t r, int64_t c, float x, float bv) {
        if (r >= g.M || c >= g.N) return;
        if (PLANES && !__builtin_isfinite(x))  // made again below
            open |= 1u << e;
        else
            write(r, c, x, alpha, bv);
    };
    auto bias_at = [&](int64_t c) { return bias != nullptr && c < g.N ? load_f32<T>(bias + c) : 0.0f; };
    auto row_of = [&](int v) { return 8 * (v / 4) + 4 * half + v % 4; };
    constexpr int OWN = 16 / S::WK;
    if constexpr (S::WK > 1) {
        // The waves that shared a 32x32 tile's contraction each finish 16 / WK of its registers.
        static_assert(TM == 1 && TN == 1, "one 32x32 tile per wave");
        constexpr int WAVES = S::WM * S::WN;
        float *red = reinterpret_cast<float *>(lds);
        __syncthreads();  // (the last tiles are read, and what came behind them is written)
#pragma unroll
        for (int v = 0; v < 16; ++v) red[(wave * 16 + v) * 64 + lane] = acc[0][0][0][v];
        __syncthreads();
        const int64_t c = n0 + wn * 32 + (lane & 31);
        const float bv = bias_at(c);
#pragma unroll
        for (int u = 0; u < OWN; ++u) {
            const int v = kg * OWN + u;
            float x = 0.0f;
#pragma unroll
            for (int p = 0; p < S::WK; ++p) x += red[((p * WAVES + wave % WAVES) * 16 + v) * 64 + lane];
            put_out(u, m0 + wm * 32 + row_of(v), c, x, bv);
        }
    } else {
        static_assert(TM * TN * 16 <= 32, "one bit per output of a lane");
#pragma unroll
        for (int w = 0; w < TN; ++w) {
            const int64_t c = n0 + wn * (BN / S::WN) + w * 32 + (lane & 31);
            const float bv = bias_at(c);
#pragma unroll
            for (int u = 0; u < TM; ++u)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    put_out((w * TM + u) * 16 + v, m0 + wm * (BM / S::WM) + u * 32 + row_of(v), c, acc[0][u][w][v], bv);
        }
    }
    if constexpr (PLANES) {
        while (open != 0) {
            const int e = __ffs(open) - 1, v = S::WK > 1 ? kg * OWN + e : e % 16, u = S::WK > 1 ? 0 : e / 16 % TM,
                      w = S::WK > 1 ? 0 : e / 16 / TM;
            open &= open - 1;
            const int64_t r = m0 + wm * (BM / S::WM) + u * 32 + row_of(v), c = n0 + wn * (BN / S::WN) + w * 32 + (lane & 31);
            write(r, c, plain_dot<T, AMODE, BMODE>(g, r, c, k_begin, k_end), g.alpha, bias_at(c));
        }
    }
}

// One launch for what a pass computes from one activation: `sketch_blocks` tiles of the sketch
// product (first: they are the long ones), `colsum_blocks` column blocks of the bias gradient and
// the tiles of the plain product.  Any of the three may be absent.
// (The operand of the sketch product is the plain product's A.  bf16: 128 registers, so that two work-groups share a compute unit;
// with the 133 that the compiler takes otherwise the backward launch of 3000 x 768 -> 1001, k = 300, is 46 us instead of 32.  The Gaussian
// forms for rows of 2^22 elements and more, 147 otherwise, have 9 and 13 of them in scratch memory and are faster for the bound too:
// backward 64 x 2^22 -> 8, k = 4, 2.8 ms instead of 4.0, forward 300 x 2^22 -> 8 60.7 instead of 62.2.)
template <typename T, typename S, typename SS, int SKETCH, int BMODE, int MODE_A, int MODE_B>
__global__ void __launch_bounds__(kPlainThreads, sizeof(T) == 2 ? 4 : 2) plain_pass_kernel(PlainArgs ga, PlainArgs gs, ColsumArgs gc, int plain_blocks,
                                                                   int sketch_blocks, int colsum_blocks) {
    constexpr int BA = PlainTile<T, S, PA_K, BMODE>::LDS_BYTES, BS = PlainTile<T, SS, SKETCH, PB_N>::LDS_BYTES;
    constexpr int BYTES = (BA > BS ? BA : BS) > kColsumLdsFloats * 4 ? (BA > BS ? BA : BS) : kColsumLdsFloats * 4;
    __shared__ __attribute__((aligned(16))) unsigned char lds[BYTES];
    const int b = (int)blockIdx.x;
    if (b < sketch_blocks)
        plain_tile<T, T, SS, SKETCH, PB_N, MODE_A, MODE_A>(gs, reinterpret_cast<bf16_t *>(lds), b, sketch_blocks);
    else if (b < sketch_blocks + colsum_blocks)
        colsum_any_body<T>(gc, reinterpret_cast<float *>(lds), b - sketch_blocks, colsum_blocks);
    else
        plain_tile<T, T, S, PA_K, BMODE, MODE_A, MODE_B>(ga, reinterpret_cast<bf16_t *>(lds), b - sketch_blocks - colsum_blocks, plain_blocks);
}

// A^T B products (dW = G^T X_proj; X^T dY of the variance monitors).
template <typename T, typename Tout, typename S, int MODE_A, int MODE_B>
__global__ void __launch_bounds__(kPlainThreads) plain_tn_kernel(PlainArgs g) {
    __shared__ __attribute__((aligned(16))) unsigned char lds[PlainTile<T, S, PA_M, PB_N>::LDS_BYTES];
    plain_tile<T, Tout, S, PA_M, PB_N, MODE_A, MODE_B>(g, reinterpret_cast<bf16_t *>(lds), blockIdx.x, gridDim.x);
}

}  // namespace

}  // namespace rmm
