// Column sums of a row-major matrix, out[c] = sum_r A[r][c] (+ the old out[c]): the bias gradient
// db = dY^T 1 (Eq. 3).  One pass over A, bound by HBM.  Device body shared by the kernel of its own
// (plain.hip) and the launch it shares with dW = G^T X_proj (mfma.hip).
//
// A work-group owns LPR x 16 bytes of every row (LPR = 4: 32 bf16 or 16 fp32 columns): thread t
// (of the first 256) takes 16 bytes of rows t / LPR, t / LPR + 256 / LPR, ..., eight loads in
// flight, and keeps fp32 sums of its 8 (4) columns; the row groups of a column are then added
// through LDS in fixed order, by all 256 threads (backward with a bias gradient, 4096 x 768 -> 768, k = 410: 29.4 us; with one
// thread a column 32.1; 3001 x 520 -> 1304, k = 600: 35.2 and 37.3; fp32 2000 x 500 -> 1000, k = 200: 53.3 and 57.0).  Column blocks that share a 128-byte line of A are numbered onto one
// XCD (work-groups are dealt round-robin to the 8 XCDs, each with its own L2), so HBM sees every
// line once.  Narrow matrices take one 16-byte piece per work-group, so that enough work-groups
// exist to pull the matrix in.  The result does not depend on the size of the work-group that runs
// the body (threads beyond the first 256 only take part in the barrier).
#pragma once
#include "common.hpp"

namespace rmm {

struct ColsumArgs {
    const void *A;  // n x d, 16-byte aligned, d a multiple of 16 bytes
    void *out;      // d
    int64_t n, d;
    int accumulate;
    int lpr;        // 16-byte pieces of a row per work-group: 4 or 1 (colsum_lpr); 0: element by element
};

inline bool colsum_wide_ok(const void *A, int64_t d, int64_t elem_bytes) {  // 16-byte loads apply
    return (d * elem_bytes) % 16 == 0 && (reinterpret_cast<uintptr_t>(A) & 15u) == 0;
}
constexpr int kColsumLdsFloats = 256 * 9 + 4 * 32;  // 256 row groups x (8 columns + 1), the larger of the two forms, and the waves' sums

// `lds` holds kColsumLdsFloats floats; block `blk` of `blocks`.
template <typename T>
__device__ __forceinline__ void colsum_body(const ColsumArgs &g, float *lds, int64_t blk, int64_t blocks) {
    constexpr int VEC = 16 / (int)sizeof(T), U = 8;
    const T *A = reinterpret_cast<const T *>(g.A);
    T *out = reinterpret_cast<T *>(g.out);
    const int tid = threadIdx.x, LPR = g.lpr, BC = VEC * LPR, RPP = 256 / LPR, PITCH = BC + 1;
    {
        const int64_t per = blocks / 8, rem = blocks % 8, x = blk % 8, r = blk / 8;
        blk = x * per + (x < rem ? x : rem) + r;
    }
    if (tid < 256) {
        const int cq = tid % LPR, rg = tid / LPR;
        const int64_t c = blk * BC + cq * VEC;
        float acc[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[e] = 0.0f;
        if (c < g.d) {
            for (int64_t r0 = rg; r0 < g.n; r0 += (int64_t)RPP * U) {
                uint4 v[U];
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (r0 + u * RPP < g.n) v[u] = *reinterpret_cast<const uint4 *>(A + (r0 + u * RPP) * g.d + c);
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (r0 + u * RPP >= g.n) break;
                    const uint32_t w[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        if constexpr (sizeof(T) == 2) {
                            acc[2 * q] += __uint_as_float(w[q] << 16);
                            acc[2 * q + 1] += __uint_as_float(w[q] & 0xFFFF0000u);
                        } else {
                            acc[q] += __uint_as_float(w[q]);
                        }
                    }
                }
            }
        }
#pragma unroll
        for (int e = 0; e < VEC; ++e) lds[rg * PITCH + cq * VEC + e] = acc[e];
    }
    __syncthreads();
    // 256 threads add VEC row groups of a column each, the lanes of a wave those of a column, a thread for each column the four waves'.
    float *waves = lds + 256 * (VEC + 1);
    if (tid < 256) {
        const int cc = tid % BC, part = tid / BC;
        float s = 0.0f;
#pragma unroll
        for (int r = 0; r < VEC; ++r) s += lds[(part * VEC + r) * PITCH + cc];
        for (int h = BC; h < 64; h <<= 1) s += __shfl_xor(s, h);
        if ((tid & 63) < BC) waves[tid / 64 * BC + cc] = s;
    }
    __syncthreads();
    const int64_t col = blk * BC + tid;
    if (tid < BC && col < g.d) {
        float s = waves[tid] + waves[BC + tid] + waves[2 * BC + tid] + waves[3 * BC + tid];
        if (g.accumulate) s += load_f32<T>(out + col);
        store_f32<T>(out + col, s);
    }
}

// The same for widths that rule out 16-byte loads: 8 columns per work-group, 32 row lanes per column with eight loads in
// flight each.  Latency bounds a thread's chain of loads (backward with a bias, 3000 x 768 -> 1001, +-1 entries: 39 us; 16
// columns and 16 lanes 63, 64 columns and 4 lanes 75).  Sixteen loads in flight cost the kernel these blocks share its third work-group per
// compute unit.
template <typename T>
__device__ __forceinline__ void colsum_narrow_body(const ColsumArgs &g, float *lds, int64_t blk, int64_t blocks) {
    constexpr int U = 8;
    const T *A = reinterpret_cast<const T *>(g.A);
    T *out = reinterpret_cast<T *>(g.out);
    {
        const int64_t per = blocks / 8, rem = blocks % 8, x = blk % 8, r = blk / 8;
        blk = x * per + (x < rem ? x : rem) + r;
    }
    const int cl = threadIdx.x & 7, rl = threadIdx.x >> 3;
    const int64_t c = blk * 8 + cl;
    float s = 0.0f;
    if (rl < 32 && c < g.d) {
        for (int64_t r = rl; r < g.n; r += 32 * U) {
            float v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = load_f32<T>(A + min(r + 32 * u, g.n - 1) * g.d + c);
#pragma unroll
            for (int u = 0; u < U; ++u) s += r + 32 * u < g.n ? v[u] : 0.0f;
        }
    }
    if (rl < 32) lds[rl * 9 + cl] = s;
    __syncthreads();
    if (rl == 0 && c < g.d) {
        float t = 0.0f;
#pragma unroll
        for (int r = 0; r < 32; ++r) t += lds[r * 9 + cl];
        if (g.accumulate) t += load_f32<T>(out + c);
        store_f32<T>(out + c, t);
    }
}

template <typename T>
__device__ __forceinline__ void colsum_any_body(const ColsumArgs &g, float *lds, int64_t blk, int64_t blocks) {
    if (g.lpr == 0)
        colsum_narrow_body<T>(g, lds, blk, blocks);
    else
        colsum_body<T>(g, lds, blk, blocks);
}

}  // namespace rmm
