// Variance monitors (Section 2.3: Lemma 2.1, Lemma 2.2, Theorem 2.3): the reductions over
// X (n x d_in) and dY (n x d_out) that the closed forms need, and the closed forms themselves.
//
//   row_norms_body       one pass over X and dY: |X|_F^2, |dY|_F^2, sum_k |x_k|^2 |y_k|^2
//                        (one wave per token row, 16-byte loads, wave-level reduction), as a kernel
//                        of its own or, on the bf16 path, in the launch of X^T dY
//   sumsq_kernel         |A|_F^2 of an fp32 buffer (the fp32 path materialises X^T dY)
//   variance_finalize    fixed-order fp64 sums of the per-block partials, then D^2_SGD,
//                        D^2_RMM, alpha
// |X^T dY|_F^2 on the bf16 path comes from the MFMA kernel of mfma.hip (tile products are
// squared and summed in the epilogue, never stored).
#include "row_norms.hpp"

namespace rmm {

namespace {

template <typename T>
__global__ void __launch_bounds__(512) row_norms_kernel(RowNormArgs g) {
    __shared__ double red[8 * 3];
    row_norms_body<T>(g, red, blockIdx.x, gridDim.x);
}

__global__ void __launch_bounds__(256) sumsq_kernel(const float *__restrict__ A, int64_t elems,
                                                    double *__restrict__ part) {
    __shared__ double red[4];
    double s = 0.0;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < elems; e += (int64_t)gridDim.x * 256) {
        const double f = A[e];
        s += f * f;
    }
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// One work-group; sixteen waves read the partials (a single one waited for 3 nb / 64 loads in a row: 6.6 us
// at nb = 1024).  out[0..7] = |X|_F^2, |dY|_F^2, sum_k |x_k|^2 |y_k|^2, |X^T dY|_F^2,
// D^2_SGD (Lemma 2.1), D^2_RMM for sketch size k and the given kind (Lemma 2.2 with the sign of
// the |X^T dY|^2 term that the fourth moment of a Gaussian entry gives, minus 2 rows / k for
// Rademacher signs), alpha (Theorem 2.3), D^2_RMM as Lemma 2.2 prints it.
__global__ void __launch_bounds__(1024) variance_finalize(const double *__restrict__ rows, int nb,
                                                          const double *__restrict__ xty, int nt, int64_t n,
                                                          int64_t k, int kind, double *__restrict__ out) {
    __shared__ double red[16][4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    for (int b = tid; b < nb; b += 1024) s[0] += rows[3 * b], s[1] += rows[3 * b + 1], s[2] += rows[3 * b + 2];
    for (int t = tid; t < nt; t += 1024) s[3] += xty[t];
#pragma unroll
    for (int i = 0; i < 4; ++i) s[i] = wave_sum(s[i]);
    if (lane == 0)
#pragma unroll
        for (int i = 0; i < 4; ++i) red[wave][i] = s[i];
    __syncthreads();
    if (tid != 0) return;
    double x2 = 0.0, y2 = 0.0, rw = 0.0, p2 = 0.0;
    for (int w = 0; w < 16; ++w) x2 += red[w][0], y2 += red[w][1], rw += red[w][2], p2 += red[w][3];
    const double B = (double)n, kk = (double)k;
    out[0] = x2, out[1] = y2, out[2] = rw, out[3] = p2;
    out[4] = n > 1 ? B / (B - 1.0) * rw - p2 / (B - 1.0) : 0.0;
    out[5] = (x2 * y2 + p2 - (kind == 1 ? 2.0 * rw : 0.0)) / kk;
    out[6] = (x2 > 0.0 && y2 > 0.0) ? p2 / (x2 * y2) : 0.0;
    out[7] = (x2 * y2 - p2) / kk;
}

}  // namespace

int sumsq_blocks(int64_t elems) {
    const int64_t b = (elems + 255) / 256;
    return (int)(b < 1024 ? b : 1024);
}

template <typename T>
hipError_t launch_row_norms(const T *X, const T *Y, int64_t n, int64_t d_in, int64_t d_out, double *part,
                            hipStream_t stream) {
    constexpr int PER = 16 / sizeof(T);
    const RowNormArgs g{X, Y, n, d_in, d_out, d_in % PER == 0 && d_out % PER == 0 ? 1 : 0, part};
    row_norms_kernel<T><<<row_norm_blocks(n), 512, 0, stream>>>(g);
    return hipGetLastError();
}

hipError_t launch_sumsq(const float *A, int64_t elems, double *part, hipStream_t stream) {
    sumsq_kernel<<<sumsq_blocks(elems), 256, 0, stream>>>(A, elems, part);
    return hipGetLastError();
}

hipError_t launch_variance_finalize(const double *rows, int nb, const double *xty, int nt, int64_t n, int64_t k,
                                    int kind, double *out, hipStream_t stream) {
    variance_finalize<<<1, 1024, 0, stream>>>(rows, nb, xty, nt, n, k, kind, out);
    return hipGetLastError();
}

template hipError_t launch_row_norms<float>(const float *, const float *, int64_t, int64_t, int64_t, double *,
                                            hipStream_t);
template hipError_t launch_row_norms<bf16_t>(const bf16_t *, const bf16_t *, int64_t, int64_t, int64_t, double *,
                                             hipStream_t);

}  // namespace rmm
