// Row norms of the variance monitors (variance.hip): device body shared by the kernel of its own and
// the launch it shares with X^T dY (mfma.hip).
#pragma once
#include "common.hpp"

namespace rmm {

// part[3*b .. 3*b+2] = (sum |x_k|^2, sum |y_k|^2, sum |x_k|^2 |y_k|^2) over the rows of block b.
struct RowNormArgs {
    const void *X, *Y;
    int64_t n, d_in, d_out;
    int vec;  // 16-byte loads apply to both
    double *part;
};

namespace {

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Sum of squares of one row, spread over the 64 lanes of a wave.
template <typename T>
__device__ __forceinline__ float row_sumsq(const T *row, int64_t d, int lane, bool vec) {
    float s = 0.0f;
    if (vec) {
        constexpr int PER = 16 / sizeof(T);  // elements per 16-byte load
        for (int64_t c = (int64_t)lane * PER; c < d; c += 64 * PER) {
            const uint4 q = *reinterpret_cast<const uint4 *>(row + c);
            if constexpr (sizeof(T) == 2) {
                const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float lo = __uint_as_float(w[i] << 16), hi = __uint_as_float(w[i] & 0xFFFF0000u);
                    s += lo * lo + hi * hi;
                }
            } else {
                const float f[4] = {__uint_as_float(q.x), __uint_as_float(q.y), __uint_as_float(q.z),
                                    __uint_as_float(q.w)};
#pragma unroll
                for (int i = 0; i < 4; ++i) s += f[i] * f[i];
            }
        }
    } else {
        for (int64_t c = lane; c < d; c += 64) {
            const float f = load_f32<T>(row + c);
            s += f * f;
        }
    }
    return wave_sum(s);
}

// Block `blk` of `blocks`; one wave per token row, the waves of a work-group take turns with those of all.
// `red` holds 3 doubles per wave.
template <typename T>
__device__ __forceinline__ void row_norms_body(const RowNormArgs &g, double *red, int64_t blk, int64_t blocks) {
    const T *X = reinterpret_cast<const T *>(g.X), *Y = reinterpret_cast<const T *>(g.Y);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = (int)(blockDim.x >> 6);
    double ax = 0.0, ay = 0.0, ar = 0.0;
    for (int64_t r = blk * waves + wave; r < g.n; r += blocks * waves) {
        const float sx = row_sumsq<T>(X + r * g.d_in, g.d_in, lane, g.vec != 0);
        const float sy = row_sumsq<T>(Y + r * g.d_out, g.d_out, lane, g.vec != 0);
        ax += sx, ay += sy, ar += (double)sx * (double)sy;
    }
    if (lane == 0) red[3 * wave] = ax, red[3 * wave + 1] = ay, red[3 * wave + 2] = ar;
    __syncthreads();
    if (threadIdx.x < 3) {
        double t = 0.0;
        for (int w = 0; w < waves; ++w) t += red[3 * w + threadIdx.x];
        g.part[3 * blk + threadIdx.x] = t;
    }
}

}  // namespace

}  // namespace rmm
