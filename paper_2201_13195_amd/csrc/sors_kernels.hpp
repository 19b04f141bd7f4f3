// Device code of the SORS sketch kind's strip kernel (see sors.hip for what it computes), kept in a
// header because it also runs inside the paired launches of a layer pass.
#pragma once
#include "common.hpp"
#include "mfma_frag.hpp"

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
__host__ __device__ constexpr int strip_phys(int t) { return t + (t >> 4) + 2 * (t >> 7); }

// ---------------------------------------------------------------------------------------------
// The kernel that serves the layer's shapes: strips of 8 columns (one 16-byte load per token row,
// the widest strip whose fp32 copy fits in LDS next to a second one), tokens taken in
// chunks of CH = 2^LC.  The transform factors over the chunks,
//
//   out[j] = sum_chunks (-1)^popcount(hi(r_j) AND chunk) * T_chunk[lo(r_j)],
//   T_chunk = the CH-point transform of the chunk's signed tokens,
//
// so a work-group runs one CH-point transform per chunk in the same LDS buffer and adds the
// selected entries into per-thread accumulators (k <= 2048, or 8192 with sixteen waves), with
// the next chunk's rows already on their way from memory.  With a single chunk (CH >= n_pad) the
// selected rows are written directly and k is not limited.
//
// A chunk's index bits, lowest first, each wave on tokens of its own as long as it can: five on the matrix pipes (the 32 x 32
// Walsh-Hadamard matrix times 32 tokens of 32 columns; the products are exact and the sums fp32), where the rows go as they are,
// bf16 with their signs, through LDS into transposed fragments; one between the halves of two registers' lanes; tiles against tiles;
// one between lanes 8 apart; then all through LDS as fp32, and the waves' bits in one pass, 16 bytes of a token at a time.  With
// every bit after the top three in two LDS passes of vector additions the vector units were busy for 54 % of the time and
// LDS for 41: 970 vector instructions a wave and chunk, 600 now, and twice the waves resident (16384 x 4096, k = 1638: 61 -> 51 us,
// 16384 x 1024 39 -> 26, 4096 x 4096, k = 4000 44 -> 31, 4096 x 768, k = 410 11.9 -> 9.1).
// LDS layout: two halves (columns 0-3, 4-7) of float4 slots, token t at slot strip_phys(t): the pads keep the sixteen-byte
// accesses, and the four-byte ones of lanes that differ in column, token bits 0 and 2, strip and upper half, on banks of their own.
//
// A backward pass with a bias gradient takes the column sums of dY here, where every element passes through registers anyway (StripSums):
// two instructions per element, ten lane exchanges at the end.  It saves the later launch its read of dY (16384 x 1024 -> 1024, k =
// 1638: backward without the bias gradient 66 us, with it 69; in a launch of its own 19 us more).  A form of its own: with a branch on
// the argument the strips without sums went from 78 us to 105 at 8192 x 4096.
template <int LC>
struct StripShape {
    static constexpr int CH = 1 << LC, SLOTS = strip_phys(CH);
    static constexpr int PLANE = SLOTS + 4, REGION = 2 * PLANE + 2;  // float4 slots of half a strip and of a strip
    static_assert(LC >= 9 && LC <= 11, "chunks of 512 .. 2048 tokens");
};

// Rows t, t + LPW, .. of a strip, 16 bytes from `off` on in each lane.  Buffer loads: a row beyond the tokens lies outside the
// descriptor's range (one for each load) and reads as zero, so there is no branch between the loads and the compiler can count
// them: with one it waited for the next chunk's rows in front of this chunk's transform.
template <int LPW, int R0>
__device__ __forceinline__ void strip_rows(const SorsArgs &g, int64_t t, uint32_t off, sors_u32x4_t (&raw)[R0]) {
#pragma unroll
    for (int i = 0; i < R0; ++i) {
        const int64_t t0 = t + i * LPW, rows = min((int64_t)LPW, g.n - t0);
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<bf16_t *>(g.A + t0 * g.d), (short)0, __builtin_amdgcn_readfirstlane((int)((rows > 0 ? rows : 0) * g.d * 2)), 0x00020000);
        raw[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, off, 0, 0);
    }
}

// The column sums of a strip, in an order of additions that depends on CH alone and not on how the waves share the strip, so that
// paired, separate and column-sum launches give the same bits: of 128 tokens of a chunk, rows r, r + 64, r + 32 and r + 96 in pairs,
// for r = 0 .. 31; this over the chunks, then over r (bits 2, 1, 0, 3, 4 of it), then over the 128-token blocks of a chunk.
// A wave has TW tokens and NPROB strips; load i of a chunk holds LPW rows from i * LPW on.
template <int CH, int TW, int NPROB>
struct StripSums {
    static constexpr int LPW = 64 / NPROB, R0 = TW / LPW, BLOCKS = TW / 128, SETS = NPROB == 2 ? BLOCKS : (BLOCKS + 1) / 2;
    static_assert(BLOCKS == 1 || BLOCKS % 2 == 0, "with one strip, lanes 32 .. 63 have every other block");
    float s[SETS][8];
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int x = 0; x < SETS; ++x)
#pragma unroll
            for (int c = 0; c < 8; ++c) s[x][c] = 0.0f;
    }
    static __device__ __forceinline__ float element(const sors_u32x4_t &raw, int c) {  // (element 2q in the low half of word q)
        return __uint_as_float(c % 2 == 0 ? raw[c / 2] << 16 : raw[c / 2] & 0xFFFF0000u);
    }
    __device__ __forceinline__ void add(const sors_u32x4_t (&raw)[R0]) {
#pragma unroll
        for (int x = 0; x < SETS; ++x)
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const int i = 4 * x;
                if constexpr (NPROB == 2) {
                    s[x][c] += (element(raw[i], c) + element(raw[i + 2], c)) + (element(raw[i + 1], c) + element(raw[i + 3], c));
                } else {  // (the halves of the lanes: rows r and r + 32)
                    const float even = element(raw[i], c) + element(raw[i + 1], c);
                    const float odd = BLOCKS == 1 ? even : element(raw[(i + 2) % R0], c) + element(raw[(i + 3) % R0], c);
                    const auto v = __builtin_amdgcn_permlane32_swap(__float_as_uint(even), __float_as_uint(odd), false, false);
                    s[x][c] += __uint_as_float(v[0]) + __uint_as_float(v[1]);
                }
                asm volatile("" : "+v"(s[x][c]));  // (now, and no copies)
            }
    }
    // The first 2 H columns of a set, over lanes that differ in bit H of the row: a lane keeps H of them.
    template <int H>
    static __device__ __forceinline__ void halve(float (&v)[8], int row) {
        const bool up = (row & H) != 0;
#pragma unroll
        for (int c = 0; c < H; ++c) {
            const float keep = up ? v[c + H] : v[c], give = up ? v[c] : v[c + H];
            v[c] = keep + __shfl_xor(give, H * NPROB);
        }
    }
    // Three exchanges leave each lane one of the eight columns, the others add; part: CH / 128 * 8 floats per strip.
    __device__ __forceinline__ void park(float *part, int wave, int lane) {
        const int prob = lane % NPROB, row = lane / NPROB % 32, half = NPROB == 2 ? 0 : lane / 32;
#pragma unroll
        for (int x = 0; x < SETS; ++x) {
            halve<4>(s[x], row), halve<2>(s[x], row), halve<1>(s[x], row);
            s[x][0] += __shfl_xor(s[x][0], 8 * NPROB);
            s[x][0] += __shfl_xor(s[x][0], 16 * NPROB);
        }
        if (row < 8 && half < BLOCKS) {
#pragma unroll
            for (int x = 0; x < SETS; ++x) part[((wave * BLOCKS + x * (3 - NPROB) + half) * NPROB + prob) * 8 + row] = s[x][0];
        }
    }
    // (behind a barrier; threads 0 .. 7 of each strip)
    static __device__ __forceinline__ void write(const SorsArgs &g, const float *part, int prob, int64_t col0, int c) {
        float x = 0.0f;
#pragma unroll
        for (int b = 0; b < CH / 128; ++b) x += part[(b * NPROB + prob) * 8 + c];
        if (g.accumulate) x += load_f32<bf16_t>(g.colsum + col0 + c);
        store_f32<bf16_t>(g.colsum + col0 + c, x);
    }
};

//
// NPROB = 2 puts two neighbouring strips into one work-group of 512 threads (thread 2r + p is
// thread r of strip p; separate LDS planes, offset by 64 bytes modulo 128 so that the interleaved
// lanes of the two strips stay on different banks): a form that shares a grid with the 512-thread
// work-groups of a plain product (one strip of 512 threads is the other, which shares compute units with them).  `block` of `blocks` numbers the work-group among those of the
// sketch product; LDS: NPROB * StripShape::REGION float4 slots and 1024 words.  With accumulators a strip's sketch columns
// may be made by `parts` work-groups, part_k (a multiple of 4) by each, up to 4 * ACC_CALLS by a thread.
template <int LC, bool ACC, int NPROB, int WAVES, bool SUMS, int ACC_CALLS = (int)kSorsAccMaxK / 4 / (64 * WAVES / NPROB)>
__device__ __forceinline__ void sors_strip_body(const SorsArgs &g, int chunks, float4 *planes_all, uint32_t *sign_words,
                                                int64_t block, int64_t blocks, int parts, int64_t part_k) {
    typedef StripShape<LC> S;
    // Threads of a strip; tokens of a wave, rows of one load of it, loads; tokens of a wave and strip in either plane, tiles of 64 of them
    constexpr int CH = S::CH, NT = 64 * WAVES / NPROB, TW = CH / WAVES, LPW = 64 / NPROB, R0 = TW / LPW, TOP = NPROB == 2 ? TW : TW / 2,
                  TILES = TOP / 64;
    static_assert(TILES >= 1 && (NPROB == 1 || WAVES >= 8), "a tile per wave");
    const int prob = NPROB == 2 ? (int)(threadIdx.x & 1) : 0;
    const int tid = NPROB == 2 ? (int)(threadIdx.x >> 1) : (int)threadIdx.x;  // thread number inside the strip
    float4 *planes = planes_all + prob * S::REGION;

    // Strips that share 128-byte lines of A should meet in one L2: work-groups are dealt round-robin
    // to the 8 XCDs, so XCD x gets a contiguous run of strips.
    int64_t group = block;
    {
        const int64_t per = blocks / 8, rem = blocks % 8, x = group % 8, r = group / 8;
        group = x * per + (x < rem ? x : rem) + r;
    }
    [[maybe_unused]] int64_t j0 = 0, j1 = g.k;  // this work-group's sketch columns (those of a strip are neighbours on an XCD, too)
    if constexpr (ACC) {
        const int64_t strip = (uint32_t)group / (uint32_t)parts;
        j0 = (group - strip * parts) * part_k, j1 = min(g.k, j0 + part_k), group = strip;
    }
    const int64_t col0 = (group * NPROB + prob) * 8;
    const bool live = col0 < g.d;  // the last work-group's second strip may not exist

    for (int c = threadIdx.x; c < chunks * (CH / 128); c += 64 * WAVES) {
        const Words4 w = philox4x32_10((uint32_t)c, kSorsSignColumn, g.st.off0, g.st.off1, g.st.key0, g.st.key1);
#pragma unroll
        for (int q = 0; q < 4; ++q) sign_words[4 * c + q] = w.w[q];
    }

    // Rows of this thread's sketch columns and their accumulators (ACC only).
    uint32_t rows[ACC ? ACC_CALLS : 1][2];  // (below 2^15: two to a register)
    auto row_of = [&](int m, int u) { return u % 2 == 0 ? rows[m][u / 2] & 0xFFFFu : rows[m][u / 2] >> 16; };
    float4 acc[ACC ? ACC_CALLS : 1][4][2];
    if constexpr (ACC) {
#pragma unroll
        for (int m = 0; m < ACC_CALLS; ++m) {
            const Words4 w = philox4x32_10((uint32_t)(j0 / 4 + tid + NT * m), kSorsRowColumn, g.st.off0, g.st.off1, g.st.key0,
                                           g.st.key1);
#pragma unroll
            for (int u = 0; u < 4; ++u) acc[m][u][0] = acc[m][u][1] = make_float4(0.f, 0.f, 0.f, 0.f);
            rows[m][0] = (w.w[0] & g.st.row_mask) | (w.w[1] & g.st.row_mask) << 16;
            rows[m][1] = (w.w[2] & g.st.row_mask) | (w.w[3] & g.st.row_mask) << 16;
        }
    }

    // Wave `wave` of the work-group loads, and transforms as far as it can alone, tokens wave * TW .. + TW - 1 of a chunk: row
    // 8 columns of it per lane, for two strips those of either in turn.
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), row = tid % LPW;
    const uint32_t off = live ? (uint32_t)((row * g.d + col0) * 2) : 0x80000000u;
    auto load_chunk = [&](int ch, sors_u32x4_t (&raw)[R0]) { strip_rows<LPW>(g, (int64_t)ch * CH + wave * TW, off, raw); };
    // The 32 x 32 Walsh-Hadamard matrix as an MFMA operand.
    bf16x8_t hadamard[2];
#pragma unroll
    for (int kh = 0; kh < 2; ++kh) {
        union {
            bf16x8_t v;
            uint16_t h[8];
        } o;
#pragma unroll
        for (int j = 0; j < 8; ++j) o.h[j] = (uint16_t)(0x3F80u | (uint32_t)(__popc((lane & 31) & (16 * kh + 8 * (lane >> 5) + j)) & 1) << 15);
        hadamard[kh] = o.v;
    }
    float4 *mine = planes_all + strip_phys(wave * TW);  // slots of the wave's tokens (of the first strip), lower half; upper half: + PLANE
    const float odd8 = (lane & 8) != 0 ? -1.0f : 1.0f;

    [[maybe_unused]] StripSums<CH, TW, NPROB> sums;
    if constexpr (SUMS) sums.clear();
    sors_u32x4_t raw[R0];
    load_chunk(0, raw);
    __syncthreads();  // sign words
    for (int ch = 0; ch < chunks; ++ch) {
        // The chunk's rows with their signs, as they are, into the wave's part of LDS: 16 bytes per row, in the plane that lane bit 3
        // of a transposed read picks (the upper half of its tokens; the strip, if there are two).
#pragma unroll
        for (int i = 0; i < R0; ++i) {
            const int t = ch * CH + wave * TW + i * LPW + row;
            const int flip = (int)(sign_words[t >> 5] << (31 - (t & 31))) >> 31;
            asm volatile("" : "+v"(raw[i]));  // (unpacked here: not before, in twice the registers)
            sors_u32x4_t w;
#pragma unroll
            for (int q = 0; q < 4; ++q) w[q] = raw[i][q] ^ ((uint32_t)flip & 0x80008000u);
            *reinterpret_cast<sors_u32x4_t *>(mine + (NPROB == 2 ? prob : i * LPW / TOP) * S::PLANE + i * LPW % TOP + row) = w;
        }
        if constexpr (SUMS) sums.add(raw);  // (while the rows go to LDS)
        if constexpr (ACC) load_chunk(ch + 1, raw);  // arrives while this chunk is transformed (past the end: zeros)
        asm volatile("" ::: "memory");  // (the wave's own LDS accesses keep their order)
        // Index bits 0 .. 4: the matrix times 32 tokens of 32 (group of 32 tokens, column) pairs a tile.
        f32x16_t acc16[TILES];
#pragma unroll
        for (int q = 0; q < TILES; ++q) {
#pragma unroll
            for (int v = 0; v < 16; ++v) acc16[q][v] = 0.0f;
#pragma unroll
            for (int kh = 0; kh < 2; ++kh) {
                const int i = lane & 15, blk = lane >> 4;
                const char *p = reinterpret_cast<const char *>(mine + ((i >> 1) & 1) * S::PLANE + 32 * (2 * q + (blk & 1)) + 16 * kh + 8 * (blk >> 1) + (i >> 2)) + (i & 1) * 8;
                typedef __attribute__((address_space(3))) s16x4_t *lds_ptr_t;
                const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(p));
                const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(p + 64));
                union {
                    s16x8_t s;
                    bf16x8_t v;
                } b;
                b.s = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                acc16[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(hadamard[kh], b.v, acc16[q], 0, 0, 0);
            }
        }
        // The other bits, in ascending order, which does not depend on WAVES or NPROB.
        // Bit 5, in lane bit 4: registers v and v + 1 (bit 0) exchange halves of their lanes, sum and difference follow.
        // Afterwards lane bit 4 is bit 0, and the lowest bit of v is bit 5.
#pragma unroll
        for (int q = 0; q < TILES; ++q)
#pragma unroll
            for (int v = 0; v < 16; v += 2) {
                const auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc16[q][v]), __float_as_uint(acc16[q][v + 1]), false, false);
                const float a = __uint_as_float(x[0]), b = __uint_as_float(x[1]);
                acc16[q][v] = a + b;
                acc16[q][v + 1] = a - b;
            }
        // Tiles: register with register.
#pragma unroll
        for (int h = 1; h < TILES; h <<= 1)
#pragma unroll
            for (int q = 0; q < TILES; ++q)
                if ((q & h) == 0) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const float a = acc16[q][v], b = acc16[q + h][v];
                        acc16[q][v] = a + b;
                        acc16[q + h][v] = a - b;
                    }
                }
        // The upper half of the wave's tokens, with one strip, in lane bit 3: in lanes that have it the result comes out negated
        // (store_row puts that right).
        if constexpr (NPROB == 1)
#pragma unroll
            for (int q = 0; q < TILES; ++q)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const float other = __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(acc16[q][v]), 0x128, 0xF, 0xF, true));  // row_ror:8
                    acc16[q][v] = fmaf(other, odd8, acc16[q][v]);
                }
        {
            asm volatile("" ::: "memory");
            const int low = ((lane >> 4) & 1) + 4 * (lane >> 5), top = (lane >> 3) & 1;
            float *p = reinterpret_cast<float *>(mine + low + top * (NPROB == 2 ? S::REGION : strip_phys(TOP)) + ((lane >> 2) & 1) * S::PLANE) + (lane & 3);
#pragma unroll
            for (int q = 0; q < TILES; ++q)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int high = 2 * ((v >> 1) & 1) + 8 * (v >> 2) + 32 * (v & 1) + 64 * q;
                    p[4 * strip_phys(high)] = acc16[q][v];
                }
        }
        __syncthreads();
        // The waves' bits, 16 bytes of a token at a time (8 or 4 where that leaves threads without one).
        {
            constexpr int E = 8 * TW / NT < 4 ? 8 * TW / NT : 4;
            typedef float vec_t __attribute__((ext_vector_type(E)));
            float *strip = reinterpret_cast<float *>(planes_all + (int)threadIdx.x / NT * S::REGION);
#pragma unroll
            for (int item = (int)threadIdx.x % NT; item < 8 / E * TW; item += NT) {
                const int h = item / (4 / E * TW), t = item / (4 / E) % TW;
                vec_t *p = reinterpret_cast<vec_t *>(strip + 4 * (h * S::PLANE + strip_phys(t)) + item % (4 / E) * E);
                vec_t v[WAVES];
#pragma unroll
                for (int w = 0; w < WAVES; ++w) v[w] = p[4 / E * strip_phys(w * TW)];
#pragma unroll
                for (int b = 1; b < WAVES; b <<= 1)
#pragma unroll
                    for (int w = 0; w < WAVES; ++w)
                        if ((w & b) == 0) {
                            const vec_t x = v[w], y = v[w + b];
                            v[w] = x + y;
                            v[w + b] = x - y;
                        }
#pragma unroll
                for (int w = 0; w < WAVES; ++w) p[4 / E * strip_phys(w * TW)] = v[w];
            }
        }
        __syncthreads();
        if constexpr (ACC) {
#pragma unroll
            for (int m = 0; m < ACC_CALLS; ++m) {
                if (j0 + 4 * (wave * (64 / NPROB) + NT * m) >= j1) continue;  // (a wave without sketch columns)
                if constexpr (SUMS)  // (their places are found anew for every chunk: kept, in front of the loop, they spill registers)
                    asm volatile("" : "+v"(rows[m][0]), "+v"(rows[m][1]));
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const uint32_t r = row_of(m, u);
                    const int at = strip_phys((int)(r & (CH - 1)));
                    const float sgn = (__popc((r >> LC) & (uint32_t)ch) & 1) ? -1.0f : 1.0f;
                    const float4 a = planes[at], b = planes[S::PLANE + at];
                    acc[m][u][0].x += sgn * a.x, acc[m][u][0].y += sgn * a.y, acc[m][u][0].z += sgn * a.z, acc[m][u][0].w += sgn * a.w;
                    acc[m][u][1].x += sgn * b.x, acc[m][u][1].y += sgn * b.y, acc[m][u][1].z += sgn * b.z, acc[m][u][1].w += sgn * b.w;
                }
            }
            __syncthreads();  // the next chunk overwrites the planes
        }
    }

    if constexpr (ACC)  // (the last request, past the end, ends here: left open, the compiler waits for it in the loop of the tile that shares the kernel)
#pragma unroll
        for (int i = 0; i < R0; ++i) asm volatile("" ::"v"(raw[i]));
    float *part = reinterpret_cast<float *>(sign_words);  // (the signs are behind a barrier)
    if constexpr (SUMS) sums.park(part, wave, lane);

    auto store_row = [&](int64_t j, uint32_t r, const float4 &a, const float4 &b) {
        const float alpha = NPROB == 1 && (r & (uint32_t)TOP) != 0 ? -g.alpha : g.alpha;
        sors_u32x4_t o;
        o.x = (uint32_t)f32_to_bf16(alpha * a.x) | ((uint32_t)f32_to_bf16(alpha * a.y) << 16);
        o.y = (uint32_t)f32_to_bf16(alpha * a.z) | ((uint32_t)f32_to_bf16(alpha * a.w) << 16);
        o.z = (uint32_t)f32_to_bf16(alpha * b.x) | ((uint32_t)f32_to_bf16(alpha * b.y) << 16);
        o.w = (uint32_t)f32_to_bf16(alpha * b.z) | ((uint32_t)f32_to_bf16(alpha * b.w) << 16);
        if (live) *reinterpret_cast<sors_u32x4_t *>(g.out + j * g.d + col0) = o;
    };
    if constexpr (ACC) {
#pragma unroll
        for (int m = 0; m < ACC_CALLS; ++m)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int64_t j = j0 + 4 * (int64_t)(tid + NT * m) + u;
                if (j < j1) store_row(j, row_of(m, u), acc[m][u][0], acc[m][u][1]);
            }
    } else {
        for (int64_t q = tid; q < (g.k + 3) / 4; q += NT) {
            const Words4 w = philox4x32_10((uint32_t)q, kSorsRowColumn, g.st.off0, g.st.off1, g.st.key0, g.st.key1);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int64_t j = 4 * q + u;
                if (j >= g.k) break;
                const uint32_t r = w.w[u] & g.st.row_mask;
                const int at = strip_phys((int)r);
                store_row(j, r, planes[at], planes[S::PLANE + at]);
            }
        }
    }
    if constexpr (SUMS) {
        __syncthreads();
        if (tid < 8 && live && j0 == 0) sums.write(g, part, prob, col0, tid);
    }
}

}  // namespace

}  // namespace rmm
