// Device code of the SORS sketch kind's strip kernel (see sors.hip for what it computes), kept in a
// header because it also runs inside the paired launches of a layer pass.
#pragma once
#include "common.hpp"

namespace rmm {

struct SorsArgs {
    const bf16_t *A;
    bf16_t *out;
    int64_t n, d, k;
    SketchState st;
    float alpha;
    bf16_t *colsum;     // kernels with SUMS: the column sums of A (the bias gradient), d values,
    int accumulate;     // added to what is there
};

namespace {

typedef unsigned int sors_u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int sors_u32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ int sors_phys(int t) { return t + (t >> 4); }

// ---------------------------------------------------------------------------------------------
// The kernel that serves the layer's shapes: strips of 8 columns (one 16-byte load per token row,
// the widest strip whose fp32 copy fits in LDS next to a second work-group's), tokens taken in
// chunks of CH = 2^LC.  The transform factors over the chunks,
//
//   out[j] = sum_chunks (-1)^popcount(hi(r_j) AND chunk) * T_chunk[lo(r_j)],
//   T_chunk = the CH-point transform of the chunk's signed tokens,
//
// so a work-group runs one CH-point transform per chunk in the same LDS buffer and adds the
// selected entries into per-thread accumulators (k <= 2048: 8 rows x 8 columns per thread), with
// the next chunk's rows already on their way from memory.  With a single chunk (CH >= n_pad) the
// selected rows are written directly and k is not limited.  Per chunk: the top LC - 8 index bits
// in registers while loading (2^(LC-8) rows per thread), then two LDS passes of four bits each,
// 16-byte LDS accesses throughout.  LDS layout: two halves (columns 0-3, 4-7) of float4 slots,
// token t at slot t + t / 16.  A backward pass with a bias gradient takes the column sums of dY here, where every
// element passes through registers anyway: eight additions per row, ten lane exchanges at the end.  It saves the later launch
// its read of dY (16384 x 1024 -> 1024, k = 1638: backward without the bias gradient 76 us, with it 103 before and 78 now;
// 4096 x 768 -> 3072, k = 410: 60 -> 52).  A form of its own: with a branch on the argument the strips without sums went
// from 78 us to 105 at 8192 x 4096.
template <int LC>
struct StripShape {
    static constexpr int CH = 1 << LC, W0 = LC - 8, R0 = 1 << W0, SLOTS = CH + CH / 16;
    static constexpr int REGION = 2 * SLOTS + 4;  // float4 slots of one strip
    static_assert(LC >= 8 && LC <= 12, "chunks of 256 .. 4096 tokens");
};
constexpr int kSorsAccCalls = 2;                      // row-selection calls per thread with accumulators
constexpr int64_t kSorsAccMaxK = 256 * 4 * kSorsAccCalls;  // 2048

__device__ __forceinline__ void sors_butterflies4(float4 (&v)[16]) {
#pragma unroll
    for (int h = 1; h < 16; h <<= 1)
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if ((i & h) == 0) {
                const float4 a = v[i], b = v[i + h];
                v[i] = make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
                v[i + h] = make_float4(a.x - b.x, a.y - b.y, a.z - b.z, a.w - b.w);
            }
}

// Index bits SHIFT .. SHIFT+3 of the chunk-local token index, both halves.  (The sixteen slots of an item lie STEP
// apart, which the slot formula does not show the compiler: it would keep an address for each of them over the whole loop.)
template <int LC, int SHIFT>
__device__ __forceinline__ void strip_lds_pass(float4 *planes, int tid) {
    typedef StripShape<LC> S;
    static_assert(SHIFT == 0 || SHIFT == 4, "two passes");
    constexpr int VEC = S::CH / 16, STEP = SHIFT == 0 ? 1 : 17;
    for (int item = tid; item < 2 * VEC; item += 256) {
        const int h = item / VEC, b = item % VEC;
        const int low = b & ((1 << SHIFT) - 1), high = b >> SHIFT;
        float4 *p = planes + h * S::SLOTS + sors_phys((high << (SHIFT + 4)) | low);
        float4 v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = p[STEP * i];
        sors_butterflies4(v);
#pragma unroll
        for (int i = 0; i < 16; ++i) p[STEP * i] = v[i];
    }
}

//
// NPROB = 2 puts two neighbouring strips into one work-group of 512 threads (thread 2r + p is
// thread r of strip p; separate LDS planes, offset by 64 bytes modulo 128 so that the interleaved
// lanes of the two strips stay on different banks): the form that shares a grid with the 512-thread
// work-groups of a plain product.  `block` of `blocks` numbers the work-group among those of the
// sketch product; LDS: NPROB * StripShape::REGION float4 slots and 1024 words.
template <int LC, bool ACC, int NPROB, bool SUMS>
__device__ __forceinline__ void sors_strip_body(const SorsArgs &g, int chunks, float4 *planes_all, uint32_t *sign_words,
                                                int64_t block, int64_t blocks) {
    typedef StripShape<LC> S;
    constexpr int CH = S::CH, R0 = S::R0;
    const int prob = NPROB == 2 ? (int)(threadIdx.x & 1) : 0;
    const int tid = NPROB == 2 ? (int)(threadIdx.x >> 1) : (int)threadIdx.x;  // thread number inside the strip, 0 .. 255
    float4 *planes = planes_all + prob * S::REGION;

    // Strips that share 128-byte lines of A should meet in one L2: work-groups are dealt round-robin
    // to the 8 XCDs, so XCD x gets a contiguous run of strips.
    int64_t group = block;
    {
        const int64_t per = blocks / 8, rem = blocks % 8, x = group % 8, r = group / 8;
        group = x * per + (x < rem ? x : rem) + r;
    }
    const int64_t col0 = (group * NPROB + prob) * 8;
    const bool live = col0 < g.d;  // the last work-group's second strip may not exist

    for (int c = threadIdx.x; c < chunks * (CH / 128); c += 256 * NPROB) {
        const Words4 w = philox4x32_10((uint32_t)c, kSorsSignColumn, g.st.off0, g.st.off1, g.st.key0, g.st.key1);
#pragma unroll
        for (int q = 0; q < 4; ++q) sign_words[4 * c + q] = w.w[q];
    }

    // Rows of this thread's sketch columns and their accumulators (ACC only).
    uint32_t rows[ACC ? kSorsAccCalls : 1][4];
    float4 acc[ACC ? kSorsAccCalls : 1][4][2];
    if constexpr (ACC) {
#pragma unroll
        for (int m = 0; m < kSorsAccCalls; ++m) {
            const Words4 w = philox4x32_10((uint32_t)(tid + 256 * m), kSorsRowColumn, g.st.off0, g.st.off1, g.st.key0,
                                           g.st.key1);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                rows[m][u] = w.w[u] & g.st.row_mask;
                acc[m][u][0] = acc[m][u][1] = make_float4(0.f, 0.f, 0.f, 0.f);
            }
        }
    }

    // Buffer loads: a row beyond the tokens lies outside the descriptor's range (256 rows each) and reads as zero, so
    // there is no branch between the loads and the compiler can count them: with one it waited for the next chunk's rows in front of
    // this chunk's transform.
    const uint32_t off = live ? (uint32_t)((tid * g.d + col0) * 2) : 0x80000000u;
    auto load_chunk = [&](int ch, sors_u32x4_t (&raw)[R0]) {
#pragma unroll
        for (int i = 0; i < R0; ++i) {
            const int64_t t0 = (int64_t)ch * CH + i * 256, rows = min((int64_t)256, g.n - t0);
            const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<bf16_t *>(g.A + t0 * g.d), (short)0, __builtin_amdgcn_readfirstlane((int)((rows > 0 ? rows : 0) * g.d * 2)), 0x00020000);
            raw[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, off, 0, 0);
        }
    };

    float sums[SUMS ? 8 : 1];
    if constexpr (SUMS)
#pragma unroll
        for (int c = 0; c < 8; ++c) sums[c] = 0.0f;
    sors_u32x4_t raw[R0];
    load_chunk(0, raw);
    __syncthreads();  // sign words
    for (int ch = 0; ch < chunks; ++ch) {
        // first pass: the chunk's top LC - 8 index bits, in registers, signs applied on the way
        {
            float4 v[R0][2];
#pragma unroll
            for (int i = 0; i < R0; ++i) {
                const int t = ch * CH + tid + i * 256;
                const uint32_t flip = ((sign_words[t >> 5] >> (t & 31)) & 1u) << 31;
                asm volatile("" : "+v"(raw[i]));  // (unpacked here: not before, in twice the registers)
                float x[8];                      // (element 2q in the low half of word q)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    x[2 * q] = __uint_as_float(raw[i][q] << 16);
                    x[2 * q + 1] = __uint_as_float(raw[i][q] & 0xFFFF0000u);
                }
                if constexpr (SUMS) {
#pragma unroll
                    for (int c = 0; c < 8; ++c) {
                        sums[c] += x[c];
                        asm volatile("" : "+v"(sums[c]));  // (now: not after all rows, with a second copy of each)
                    }
                }
#pragma unroll
                for (int c = 0; c < 8; ++c) x[c] = __uint_as_float(__float_as_uint(x[c]) ^ flip);
                v[i][0] = make_float4(x[0], x[1], x[2], x[3]);
                v[i][1] = make_float4(x[4], x[5], x[6], x[7]);
            }
            if constexpr (ACC) load_chunk(ch + 1, raw);  // arrives while this chunk is transformed (past the end: zeros)
#pragma unroll
            for (int h = 1; h < R0; h <<= 1)
#pragma unroll
                for (int i = 0; i < R0; ++i)
                    if ((i & h) == 0) {
#pragma unroll
                        for (int e = 0; e < 2; ++e) {
                            const float4 a = v[i][e], b = v[i + h][e];
                            v[i][e] = make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
                            v[i + h][e] = make_float4(a.x - b.x, a.y - b.y, a.z - b.z, a.w - b.w);
                        }
                    }
#pragma unroll
            for (int i = 0; i < R0; ++i) {
                float4 *p = planes + sors_phys(tid) + 272 * i;  // token tid + 256 i
                p[0] = v[i][0];
                p[S::SLOTS] = v[i][1];
            }
        }
        __syncthreads();
        strip_lds_pass<LC, 4>(planes, tid);
        __syncthreads();
        strip_lds_pass<LC, 0>(planes, tid);
        __syncthreads();
        if constexpr (ACC) {
#pragma unroll
            for (int m = 0; m < kSorsAccCalls; ++m)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const uint32_t r = rows[m][u];
                    const int at = sors_phys((int)(r & (CH - 1)));
                    const float sgn = (__popc((r >> LC) & (uint32_t)ch) & 1) ? -1.0f : 1.0f;
                    const float4 a = planes[at], b = planes[S::SLOTS + at];
                    acc[m][u][0].x += sgn * a.x, acc[m][u][0].y += sgn * a.y, acc[m][u][0].z += sgn * a.z, acc[m][u][0].w += sgn * a.w;
                    acc[m][u][1].x += sgn * b.x, acc[m][u][1].y += sgn * b.y, acc[m][u][1].z += sgn * b.z, acc[m][u][1].w += sgn * b.w;
                }
            __syncthreads();  // the next chunk overwrites the planes
        }
    }

    float *wave_sums = reinterpret_cast<float *>(sign_words);  // (the signs are behind a barrier) 8 per wave and strip
    if constexpr (SUMS) {
        // Over the lanes of a strip in fixed order: three exchanges leave each lane one of the eight columns, the others add.
        const int lane = (int)threadIdx.x % 64 / NPROB;
#pragma unroll
        for (int h = 4; h > 0; h >>= 1)
#pragma unroll
            for (int c = 0; c < h; ++c) {
                const bool up = (lane & h) != 0;
                const float keep = up ? sums[c + h] : sums[c], give = up ? sums[c] : sums[c + h];
                sums[c] = keep + __shfl_xor(give, h * NPROB);
            }
#pragma unroll
        for (int h = 8; h < 64 / NPROB; h <<= 1) sums[0] += __shfl_xor(sums[0], h * NPROB);
        if (lane < 8) wave_sums[((int)threadIdx.x / 64 * NPROB + prob) * 8 + lane] = sums[0];
    }

    auto store_row = [&](int64_t j, const float4 &a, const float4 &b) {
        sors_u32x4_t o;
        o.x = (uint32_t)f32_to_bf16(g.alpha * a.x) | ((uint32_t)f32_to_bf16(g.alpha * a.y) << 16);
        o.y = (uint32_t)f32_to_bf16(g.alpha * a.z) | ((uint32_t)f32_to_bf16(g.alpha * a.w) << 16);
        o.z = (uint32_t)f32_to_bf16(g.alpha * b.x) | ((uint32_t)f32_to_bf16(g.alpha * b.y) << 16);
        o.w = (uint32_t)f32_to_bf16(g.alpha * b.z) | ((uint32_t)f32_to_bf16(g.alpha * b.w) << 16);
        if (live) *reinterpret_cast<sors_u32x4_t *>(g.out + j * g.d + col0) = o;
    };
    if constexpr (ACC) {
#pragma unroll
        for (int m = 0; m < kSorsAccCalls; ++m)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int64_t j = 4 * (int64_t)(tid + 256 * m) + u;
                if (j < g.k) store_row(j, acc[m][u][0], acc[m][u][1]);
            }
    } else {
        for (int64_t q = tid; q < (g.k + 3) / 4; q += 256) {
            const Words4 w = philox4x32_10((uint32_t)q, kSorsRowColumn, g.st.off0, g.st.off1, g.st.key0, g.st.key1);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int64_t j = 4 * q + u;
                if (j >= g.k) break;
                const int at = sors_phys((int)(w.w[u] & g.st.row_mask));
                store_row(j, planes[at], planes[S::SLOTS + at]);
            }
        }
    }
    if constexpr (SUMS) {
        __syncthreads();
        if (tid < 8 && live) {
            float x = 0.0f;
#pragma unroll
            for (int w = 0; w < 4 * NPROB; ++w) x += wave_sums[(w * NPROB + prob) * 8 + tid];
            if (g.accumulate) x += load_f32<bf16_t>(g.colsum + col0 + tid);
            store_f32<bf16_t>(g.colsum + col0 + tid, x);
        }
    }
}

}  // namespace

}  // namespace rmm
