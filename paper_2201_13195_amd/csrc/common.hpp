// Shared device helpers and the host-side launcher declarations of the library.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "launch_plans.hpp"
#include "philox.hpp"

namespace rmm {

typedef uint16_t bf16_t;  // raw bfloat16 bits

__device__ __forceinline__ float bf16_to_f32(bf16_t x) { return __uint_as_float((uint32_t)x << 16); }

// Round to nearest even; NaN stays NaN (quiet).
__device__ __forceinline__ bf16_t f32_to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (bf16_t)((u >> 16) | 0x0040u);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (bf16_t)(u >> 16);
}

template <typename T>
__device__ __forceinline__ float load_f32(const T *p);
template <>
__device__ __forceinline__ float load_f32<float>(const float *p) { return *p; }
template <>
__device__ __forceinline__ float load_f32<bf16_t>(const bf16_t *p) { return bf16_to_f32(*p); }

template <typename T>
__device__ __forceinline__ void store_f32(T *p, float v);
template <>
__device__ __forceinline__ void store_f32<float>(float *p, float v) { *p = v; }
template <>
__device__ __forceinline__ void store_f32<bf16_t>(bf16_t *p, float v) { *p = f32_to_bf16(v); }

// ---------------------------------------------------------------------------
// Host launchers (each returns the hipError_t of its launches).
// ---------------------------------------------------------------------------

// fp32-matrix kernels (plain.hip): the fp32 data path, and the bf16 shapes the bf16 MFMA path does
// not take.  One launch per call:
//   (`cut`: the token slices of the sketch product, their sums in `ws`)
//   Y = X W^T (+ bias) and X_proj = S^T X; either output may be null
template <typename T>
hipError_t launch_forward_plain(const T *X, const T *W, const T *bias, T *Y, T *X_proj, int64_t n, int64_t d_in,
                                int64_t d_out, int64_t k, int kind, SketchState st, hipStream_t stream,
                                const PlainSlices &cut, void *ws);
//   dX = dY W, G = S^T dY and dbias = dY^T 1 (+ the old dbias); any output may be null
template <typename T>
hipError_t launch_backward_plain(const T *dY, const T *W, T *dX, T *G, T *dbias, int64_t n, int64_t d_in, int64_t d_out,
                                 int64_t k, int kind, SketchState st, bool accumulate_dbias, hipStream_t stream,
                                 const PlainSlices &cut, void *ws);
//   C[m x n] = A^T B (+ the old C if `accumulate`), A[kk x m], B[kk x n]
template <typename Tin, typename Tout>
hipError_t launch_tn_plain(const Tin *A, int64_t lda, const Tin *B, Tout *C, int64_t m, int64_t n, int64_t kk, hipStream_t stream,
                           bool accumulate = false);
//   out[d] = column sums of A[n x d] (+ the old out if `accumulate`).
template <typename T>
hipError_t launch_colsum(const T *A, T *out, int64_t n, int64_t d, hipStream_t stream, bool accumulate = false);

// bf16 MFMA path (mfma.hip).  Usable when mfma_shape_ok(); `ws` for the sketch
// must hold sketch_workspace_bf16() bytes (fp32 partial sums of the token slices), in a pass those of `room` slices.
// launch_sketch_bf16 records the optional event pair around its product kernel
// alone (the sum over token slices, when there is one, comes after `ev_end`).
// (`pair_k`, if not 0: with the tiles of the pass's paired launch with a sketch of pair_k columns, for passes that launch
// their products one by one)
hipError_t launch_linear_nt_bf16(const bf16_t *X, const bf16_t *W, const bf16_t *bias, bf16_t *Y, int64_t n,
                                 int64_t d_in, int64_t d_out, int64_t pair_k, int kind, int64_t room, hipStream_t stream);
hipError_t launch_linear_nn_bf16(const bf16_t *dY, const bf16_t *W, bf16_t *dX, int64_t n, int64_t d_in,
                                 int64_t d_out, int64_t pair_k, int kind, int64_t room, hipStream_t stream);
hipError_t launch_dw_bf16(const bf16_t *G, const bf16_t *X_proj, bf16_t *dW, int64_t k, int64_t d_in, int64_t d_out,
                          hipStream_t stream, bool accumulate = false);
// dW together with db = column sums of dY (n x d_out, 16-byte aligned, d_out a multiple of 8) in
// one launch; same results as launch_dw_bf16 followed by launch_colsum, bit for bit.
hipError_t launch_dw_colsum_bf16(const bf16_t *G, const bf16_t *X_proj, bf16_t *dW, int64_t k, int64_t d_in, int64_t d_out,
                                 const bf16_t *dY, bf16_t *dbias, int64_t n, hipStream_t stream, bool accumulate = false);
// `d_other` > 0 says that the sketch product belongs to a layer pass whose plain product has an
// n x d_other output (forward: d = d_in, d_other = d_out; backward: d = d_out, d_other = d_in): the
// token slicing is then the one the paired launch of that pass uses, so that the separate and the
// paired launches give the same bits.  0 = the product on its own (rmm_sketch).  `with_dbias`: a backward
// pass that also makes the bias gradient (it may slice the tokens otherwise).
hipError_t launch_sketch_bf16(const bf16_t *A, bf16_t *out, int64_t n, int64_t d, int64_t k, int kind, SketchState st,
                              void *ws, hipStream_t stream, hipEvent_t ev_begin = nullptr,
                              hipEvent_t ev_end = nullptr, int64_t d_other = 0, bool with_dbias = false, int64_t room = kMostSlices);

// One launch for the two products of a pass that do not depend on each other: Y = X W^T (+ bias)
// with the sketch product of X (forward), dX = dY W with the sketch product of dY (backward; G is
// k x d_out), followed by the sum over the sketch's token slices.  Results are bit-identical to
// the separate launches above (same kernels, same slices).  Only where pass_pair_available() says so;
// the optional event pair brackets the paired kernel alone.
hipError_t launch_forward_pair_bf16(const bf16_t *X, const bf16_t *W, const bf16_t *bias, bf16_t *Y, bf16_t *X_proj,
                                    int64_t n, int64_t d_in, int64_t d_out, int64_t k, int kind, SketchState st, void *ws, int64_t room,
                                    hipStream_t stream, hipEvent_t ev_begin = nullptr, hipEvent_t ev_end = nullptr);
// `with_dbias`: the pass makes the bias gradient, in whichever launch.  With `dbias` this launch takes the
// column sums of dY, on the compute units its last round leaves idle; backward_pair_takes_colsum() says where that
// beats the launch of dW.
hipError_t launch_backward_pair_bf16(const bf16_t *dY, const bf16_t *W, bf16_t *dX, bf16_t *G, int64_t n, int64_t d_in,
                                     int64_t d_out, int64_t k, int kind, SketchState st, void *ws, int64_t room, hipStream_t stream,
                                     hipEvent_t ev_begin, hipEvent_t ev_end, bool with_dbias, bf16_t *dbias,
                                     bool accumulate_dbias);
bool backward_pair_takes_colsum_in(int64_t n, int64_t d_in, int64_t d_out, int64_t k, int kind, int64_t room);
bool backward_pair_takes_colsum(int64_t n, int64_t d_in, int64_t d_out, int64_t k, int kind);  // in any scratch asked for

// SORS sketch kind, bf16 (sors.hip): signs, Walsh-Hadamard transform along the tokens and row
// selection in one kernel, no workspace.  Usable when sors_fast_ok(): d a multiple of 8 and at most
// 32768 tokens (rows in 16 bits, signs in LDS); `st` made with the token count.
// `colsum`, if not null, gets the column sums of A from the same pass over it.
bool sors_fast_ok(int64_t n, int64_t d);
hipError_t launch_sors_bf16(const bf16_t *A, bf16_t *out, int64_t n, int64_t d, int64_t k, SketchState st,
                            hipStream_t stream, bf16_t *colsum = nullptr, bool accumulate = false);
// The column sums alone, with the same bits.
hipError_t launch_sors_colsum_bf16(const bf16_t *A, bf16_t *colsum, int64_t n, int64_t d, int64_t k, bool accumulate, hipStream_t stream);

// One launch for the plain product of a pass and the SORS sketch product of the same pass, where
// the plain product leaves compute units idle (mfma.hip decides, mfma_pair_sors.hip holds the
// kernels).  Same results as the separate launches, bit for bit.
bool sors_pair_available(int64_t n, int64_t d_sk, int64_t d_other, int64_t k);
// Whether the strips can have compute units of their own in that launch (what rmm_uses_paired_launch says of this kind).
bool sors_strips_among_rounds(int64_t n, int64_t d_sk, int64_t d_other, int64_t k);
hipError_t launch_forward_pair_sors_bf16(const bf16_t *X, const bf16_t *W, const bf16_t *bias, bf16_t *Y, bf16_t *X_proj,
                                         int64_t n, int64_t d_in, int64_t d_out, int64_t k, SketchState st,
                                         hipStream_t stream, hipEvent_t ev_begin = nullptr, hipEvent_t ev_end = nullptr);
hipError_t launch_backward_pair_sors_bf16(const bf16_t *dY, const bf16_t *W, bf16_t *dX, bf16_t *G, int64_t n,
                                          int64_t d_in, int64_t d_out, int64_t k, SketchState st, bf16_t *dbias,
                                          bool accumulate_dbias, hipStream_t stream, hipEvent_t ev_begin = nullptr,
                                          hipEvent_t ev_end = nullptr);

// Variance monitors (variance.hip, and the squared-norm epilogue of the MFMA kernel).
//   part[3*b..] = per-block (sum |x_k|^2, sum |y_k|^2, sum |x_k|^2 |y_k|^2); row_norm_blocks(n) blocks.
template <typename T>
hipError_t launch_row_norms(const T *X, const T *Y, int64_t n, int64_t d_in, int64_t d_out, double *part,
                            hipStream_t stream);
//   part[b] = per-block sum of squares of an fp32 buffer; sumsq_blocks(elems) blocks.
int sumsq_blocks(int64_t elems);
hipError_t launch_sumsq(const float *A, int64_t elems, double *part, hipStream_t stream);
//   part[t] = sum of squares of tile t of X^T dY (d_in x d_out), bf16 MFMA path; xty_sumsq_tiles() tiles;
//   rows = the row norms (part of launch_row_norms), in the same launch.
hipError_t launch_xty_norms_bf16(const bf16_t *X, const bf16_t *dY, double *part, double *rows, int64_t n, int64_t d_in,
                                 int64_t d_out, int64_t room, hipStream_t stream);
hipError_t launch_variance_finalize(const double *rows, int nb, const double *xty, int nt, int64_t n, int64_t k,
                                    int kind, double *out, hipStream_t stream);

hipError_t launch_debug_philox(SketchState st, uint32_t c0, uint32_t c1, int64_t ncalls, uint32_t *out,
                               hipStream_t stream);
hipError_t launch_debug_sketch_tile(int kind, SketchState st, int64_t i0, int64_t j0, int64_t rows, int64_t cols,
                                    float *out, hipStream_t stream);

}  // namespace rmm
