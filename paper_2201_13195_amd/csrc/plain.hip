// Host side of the fp32 kernels (plain_kernels.hpp): launches (launch_plans.hpp: tile shapes, slices), and the small kernels
// that go with them (column sums on their own, the generator test hooks).
#include <type_traits>

#include "plain_pass.hpp"

namespace rmm {

namespace {

template <typename T>
__global__ void __launch_bounds__(256) colsum_kernel(ColsumArgs g) {
    __shared__ __attribute__((aligned(16))) float lds[kColsumLdsFloats];
    colsum_any_body<T>(g, lds, blockIdx.x, gridDim.x);
}

template <typename T>
ColsumArgs colsum_args(const T *A, T *out, int64_t n, int64_t d, bool accumulate, int *blocks) {
    const bool wide = colsum_wide_ok(A, d, sizeof(T));
    *blocks = (int)(wide ? colsum_blocks(d, sizeof(T)) : colsum_narrow_blocks(d));
    return ColsumArgs{A, out, n, d, accumulate ? 1 : 0, wide ? colsum_lpr(d, sizeof(T)) : 0};
}

template <typename T>
hipError_t launch_pass(PlainLaunch &p, bool has_plain, bool has_sketch, bool b_rows_k, int mode, int cfg, hipStream_t stream) {
    if (mode == 0)
        cfg = PLAIN_TINY;
    else if (cfg < 0)
        cfg = has_plain ? plain_cfg(sizeof(T), p.ga.M, p.ga.N, b_rows_k) : PLAIN_MID;
    p.cfg = has_plain || mode == 0 ? cfg : PLAIN_MID;
    p.plain_blocks = has_plain ? (int)plain_tiles(p.cfg, p.ga.M, p.ga.N) : 0;
    p.sketch_blocks = 0;
    p.sketch_small = false;
    if (has_sketch) {
        p.sketch_small = mode == 0 || (p.gs.slices <= 1 && plain_sketch_small(cfg, p.gs.M, p.gs.N));
        p.sketch_blocks = (int)tiles_of(p.gs.M, p.gs.N, 32, p.sketch_small ? 32 : 128) * (p.gs.slices > 1 ? p.gs.slices : 1);
    }
    if constexpr (sizeof(T) == 2) {
        const bool a16 = rows_on_16(has_plain ? p.ga.lda : p.gs.ldb), b16 = rows_on_16(has_plain ? p.ga.ldb : p.gs.ldb);
        if (mode != 0 && !b_rows_k && a16 && b16) return launch_forward_pass_bf16x8(p, stream);
        if (mode != 0 && b_rows_k && (!has_plain ? a16 : a16 && !b16)) return launch_backward_pass_bf16x8_(p, stream);
        if (mode != 0 && b_rows_k && !a16 && b16) return launch_backward_pass_bf16_x8(p, stream);
        return mode == 0 ? launch_plain_pass_far_bf16(p, b_rows_k, stream) : launch_plain_pass_bf16(p, b_rows_k, stream);
    } else {
        return mode == 0   ? launch_plain_pass_far_f32(p, b_rows_k, stream)
               : mode == 4 ? launch_plain_pass_f32x4(p, b_rows_k, stream)
                           : launch_plain_pass_f32(p, b_rows_k, stream);
    }
}

template <typename T>
PlainArgs sketch_args(const T *A, T *out, int64_t n, int64_t d, int64_t k, int kind, SketchState st, const PlainSlices &cut, void *ws) {
    PlainArgs g{};
    g.B = A, g.ldb = d, g.C = cut.slices > 1 ? ws : (void *)out, g.ldc = cut.ld != 0 ? cut.ld : d, g.M = k, g.N = d, g.K = n, g.alpha = 1.0f / sqrtf((float)k);
    g.kind = kind, g.st = st;
    g.slices = cut.slices, g.k_chunk = cut.slices > 1 ? cut.chunk : n, g.split_stride = cut.stride;
    return g;
}

// out = alpha * the sum of the slices' sums, in their order.  (Rows of a multiple of 8 values: what lies behind a row's
// end is summed too, and used by nobody.)
__global__ void __launch_bounds__(256) reduce_slices_kernel(const float *__restrict__ part, bf16_t *__restrict__ out, int64_t elems,
                                                            int slices, float alpha) {
    const int64_t e = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (e >= elems) return;
    float4 s = *reinterpret_cast<const float4 *>(part + e);
#pragma unroll 8
    for (int z = 1; z < slices; ++z) {
        const float4 p = *reinterpret_cast<const float4 *>(part + z * elems + e);
        s.x += p.x, s.y += p.y, s.z += p.z, s.w += p.w;
    }
    uint2 o;
    o.x = (uint32_t)f32_to_bf16(alpha * s.x) | ((uint32_t)f32_to_bf16(alpha * s.y) << 16);
    o.y = (uint32_t)f32_to_bf16(alpha * s.z) | ((uint32_t)f32_to_bf16(alpha * s.w) << 16);
    *reinterpret_cast<uint2 *>(out + e) = o;
}

// The slices of a pass's sketch product are its last launch.
template <typename T>
hipError_t finish_slices(const PlainArgs &gs, T *out, hipStream_t stream) {
    if constexpr (sizeof(T) == 2) {
        reduce_slices_kernel<<<(unsigned)((gs.split_stride + 1023) / 1024), 256, 0, stream>>>((const float *)gs.C, out, gs.split_stride,
                                                                                              gs.slices, gs.alpha);
    }
    return hipGetLastError();
}

template <typename T, typename Tout, int MODE_A, int MODE_B>
hipError_t launch_tn(const PlainArgs &g, hipStream_t stream) {
    const int cfg = MODE_A == 0 ? PLAIN_TINY : plain_cfg(sizeof(T), g.M, g.N, true);
    const unsigned grid = (unsigned)plain_tiles(cfg, g.M, g.N);
    if constexpr (MODE_A != 0) {
        if (cfg == PLAIN_BIG) {
            plain_tn_kernel<T, Tout, PlainBig, MODE_A, MODE_B><<<grid, kPlainThreads, 0, stream>>>(g);
            return hipGetLastError();
        }
        if (cfg == PLAIN_MID) {
            plain_tn_kernel<T, Tout, PlainMid, MODE_A, MODE_B><<<grid, kPlainThreads, 0, stream>>>(g);
            return hipGetLastError();
        }
    }
    plain_tn_kernel<T, Tout, PlainTiny, MODE_A, MODE_B><<<grid, kPlainThreads, 0, stream>>>(g);
    return hipGetLastError();
}

__global__ void debug_philox_kernel(SketchState st, uint32_t c0, uint32_t c1, int64_t ncalls,
                                    uint32_t *__restrict__ out) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= ncalls) return;
    const Words4 r = philox4x32_10(c0 + (uint32_t)t, c1, st.off0, st.off1, st.key0, st.key1);
#pragma unroll
    for (int q = 0; q < 4; ++q) out[4 * t + q] = r.w[q];
}

__global__ void debug_sketch_tile_kernel(int kind, SketchState st, int64_t i0, int64_t j0, int64_t rows,
                                         int64_t cols, float *__restrict__ out) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= rows * cols) return;
    const int64_t r = e / cols, c = e % cols;
    out[e] = sketch_entry_precise(kind, st, i0 + r, j0 + c);
}

}  // namespace

template <typename T>
hipError_t launch_forward_plain(const T *X, const T *W, const T *bias, T *Y, T *X_proj, int64_t n, int64_t d_in,
                                int64_t d_out, int64_t k, int kind, SketchState st, hipStream_t stream, const PlainSlices &cut, void *ws) {
    PlainLaunch p{};
    if (Y != nullptr) {
        p.ga.A = X, p.ga.lda = d_in, p.ga.B = W, p.ga.ldb = d_in, p.ga.C = Y, p.ga.ldc = d_out, p.ga.bias = bias;
        p.ga.M = n, p.ga.N = d_out, p.ga.K = d_in, p.ga.alpha = 1.0f;
    }
    if (X_proj != nullptr) p.gs = sketch_args<T>(X, X_proj, n, d_in, k, kind, st, cut, ws);
    p.tile = cut.cfg >= 0 ? cut.tile : any_width_tile(plain_cfg(sizeof(T), n, d_out, false), n, d_out, d_in);  // (without a sketch product in the pass: Y alone)
    const hipError_t e = launch_pass<T>(p, Y != nullptr, X_proj != nullptr, false, load_mode(sizeof(T), d_in, d_in), cut.cfg, stream);
    return e != hipSuccess || cut.slices <= 1 || X_proj == nullptr ? e : finish_slices<T>(p.gs, X_proj, stream);
}

template <typename T>
hipError_t launch_backward_plain(const T *dY, const T *W, T *dX, T *G, T *dbias, int64_t n, int64_t d_in, int64_t d_out,
                                 int64_t k, int kind, SketchState st, bool accumulate_dbias, hipStream_t stream, const PlainSlices &cut,
                                 void *ws) {
    PlainLaunch p{};
    if (dX != nullptr) {
        p.ga.A = dY, p.ga.lda = d_out, p.ga.B = W, p.ga.ldb = d_in, p.ga.C = dX, p.ga.ldc = d_in;
        p.ga.M = n, p.ga.N = d_in, p.ga.K = d_out, p.ga.alpha = 1.0f;
    }
    if (G != nullptr) p.gs = sketch_args<T>(dY, G, n, d_out, k, kind, st, cut, ws);
    if (dbias != nullptr) p.gc = colsum_args<T>(dY, dbias, n, d_out, accumulate_dbias, &p.colsum_blocks);
    const hipError_t e = launch_pass<T>(p, dX != nullptr, G != nullptr, true, load_mode(sizeof(T), d_in, d_out), cut.cfg, stream);
    return e != hipSuccess || cut.slices <= 1 || G == nullptr ? e : finish_slices<T>(p.gs, G, stream);
}

template <typename Tin, typename Tout>
hipError_t launch_tn_plain(const Tin *A, int64_t lda, const Tin *B, Tout *C, int64_t m, int64_t n, int64_t kk, hipStream_t stream,
                           bool accumulate) {
    PlainArgs g{};
    g.A = A, g.lda = lda, g.B = B, g.ldb = n, g.C = C, g.ldc = n, g.M = m, g.N = n, g.K = kk, g.alpha = 1.0f;
    g.accumulate = accumulate ? 1 : 0;
    const int mode = load_mode(sizeof(Tin), m, n);
    if (mode == 0) return launch_tn<Tin, Tout, 0, 0>(g, stream);
    if constexpr (sizeof(Tin) == 4) {
        if (mode == 4) return launch_tn<Tin, Tout, 4, 4>(g, stream);
    } else if constexpr (sizeof(Tout) == 2) {  // (G has rows on 16 bytes)
        if (rows_on_16(lda)) return rows_on_16(n) ? launch_tn<Tin, Tout, 4, 4>(g, stream) : launch_tn<Tin, Tout, 4, 3>(g, stream);
    }
    return launch_tn<Tin, Tout, 3, 3>(g, stream);
}

template <typename T>
hipError_t launch_colsum(const T *A, T *out, int64_t n, int64_t d, hipStream_t stream, bool accumulate) {
    int blocks = 0;
    const ColsumArgs g = colsum_args<T>(A, out, n, d, accumulate, &blocks);
    colsum_kernel<T><<<(unsigned)blocks, 256, 0, stream>>>(g);
    return hipGetLastError();
}

hipError_t launch_debug_philox(SketchState st, uint32_t c0, uint32_t c1, int64_t ncalls, uint32_t *out,
                               hipStream_t stream) {
    debug_philox_kernel<<<(unsigned)((ncalls + 255) / 256), 256, 0, stream>>>(st, c0, c1, ncalls, out);
    return hipGetLastError();
}

hipError_t launch_debug_sketch_tile(int kind, SketchState st, int64_t i0, int64_t j0, int64_t rows, int64_t cols,
                                    float *out, hipStream_t stream) {
    const int64_t total = rows * cols;
    debug_sketch_tile_kernel<<<(unsigned)((total + 255) / 256), 256, 0, stream>>>(kind, st, i0, j0, rows, cols, out);
    return hipGetLastError();
}

#define RMM_INSTANTIATE(T)                                                                                           \
    template hipError_t launch_forward_plain<T>(const T *, const T *, const T *, T *, T *, int64_t, int64_t,         \
                                                int64_t, int64_t, int, SketchState, hipStream_t, const PlainSlices &, void *);                    \
    template hipError_t launch_backward_plain<T>(const T *, const T *, T *, T *, T *, int64_t, int64_t, int64_t,     \
                                                 int64_t, int, SketchState, bool, hipStream_t, const PlainSlices &, void *);                      \
    template hipError_t launch_tn_plain<T, T>(const T *, int64_t, const T *, T *, int64_t, int64_t, int64_t,         \
                                              hipStream_t, bool);                                                    \
    template hipError_t launch_colsum<T>(const T *, T *, int64_t, int64_t, hipStream_t, bool);
RMM_INSTANTIATE(float)
RMM_INSTANTIATE(bf16_t)
#undef RMM_INSTANTIATE
template hipError_t launch_tn_plain<bf16_t, float>(const bf16_t *, int64_t, const bf16_t *, float *, int64_t, int64_t, int64_t,
                                                   hipStream_t, bool);

}  // namespace rmm
