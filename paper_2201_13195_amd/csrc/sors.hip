// The SORS sketch kind (subsampled orthonormal matrix with random signs; the paper names the
// family in Section 2.1 and points at its O(B N log B) cost in Section 3.5 and in the future-work
// paragraph, without a construction; the one used here is stated in include/rmm.h): the token signs,
// the Walsh-Hadamard transform along the token axis and the row selection in one pass over A.
//
//   A_proj[j][c] = (1 / sqrt(k)) * sum_i (-1)^popcount(i AND r_j) * sigma_i * A[i][c]
//
// It is done by the strip kernels of sors_kernels.hpp.
#include "sors_kernels.hpp"

namespace rmm {

namespace {

// Eight waves a strip (four where a chunk has tokens for no more): two strips are resident on a compute unit, by LDS.
template <int LC>
constexpr int strip_waves() { return LC == 9 ? 4 : 8; }
template <int LC, bool ACC, int NPROB, bool SUMS>
__global__ void __launch_bounds__(64 * NPROB * strip_waves<LC>(), strip_waves<LC>() / 2) sors_strip_kernel(SorsArgs g, int chunks) {
    __shared__ float4 planes[NPROB * StripShape<LC>::REGION];
    __shared__ uint32_t sign_words[1024];  // up to 32768 tokens
    sors_strip_body<LC, ACC, NPROB, NPROB * strip_waves<LC>(), SUMS>(g, chunks, planes, sign_words, blockIdx.x, gridDim.x, 1, g.k);
}

template <int LC, bool ACC, int NPROB>
hipError_t launch_strips(const SorsArgs &g, int chunks, hipStream_t stream) {
    const unsigned grid = (unsigned)((g.d / 8 + NPROB - 1) / NPROB), threads = 64 * NPROB * strip_waves<LC>();
    if (g.colsum != nullptr)
        sors_strip_kernel<LC, ACC, NPROB, true><<<grid, threads, 0, stream>>>(g, chunks);
    else
        sors_strip_kernel<LC, ACC, NPROB, false><<<grid, threads, 0, stream>>>(g, chunks);
    return hipGetLastError();
}

// Two strips to a work-group where some compute unit has two anyway: a row is then 32 bytes of a line instead of 16, and half as many
// lines go from L2 to the compute units, which at 16384 x 4096 is what the strips wait for (58 -> 51 us; 8192 x 4096 32.5 -> 28,
// 4096 x 3072 17.0 -> 15.4; at 16384 x 1024, where every strip has a compute unit of its own, 26 -> 36).
template <int LC, bool ACC>
hipError_t launch_strip(const SorsArgs &g, int chunks, hipStream_t stream) {
    if constexpr (LC == 11)
        if (g.d / 8 > 256) return launch_strips<LC, ACC, 2>(g, chunks, stream);
    return launch_strips<LC, ACC, 1>(g, chunks, stream);
}

// The column sums alone, as the strips take them: for a pass whose bias gradient is to be timed on its own.
template <int LC>
__global__ void __launch_bounds__(64 * strip_waves<LC>()) sors_colsum_kernel(SorsArgs g, int chunks) {
    constexpr int CH = 1 << LC, TW = CH / strip_waves<LC>();
    typedef StripSums<CH, TW, 1> Sums;
    __shared__ float part[CH / 128 * 8];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int64_t col0 = (int64_t)blockIdx.x * 8;
    const uint32_t off = (uint32_t)((lane * g.d + col0) * 2);
    Sums sums;
    sums.clear();
    for (int ch = 0; ch < chunks; ++ch) {
        sors_u32x4_t raw[Sums::R0];
        strip_rows<64>(g, (int64_t)ch * CH + wave * TW, off, raw);
        sums.add(raw);
    }
    sums.park(part, wave, lane);
    __syncthreads();
    if (threadIdx.x < 8) sums.write(g, part, 0, col0, (int)threadIdx.x);
}

template <int LC>
hipError_t launch_colsum_strips(const SorsArgs &g, int chunks, hipStream_t stream) {
    sors_colsum_kernel<LC><<<(unsigned)(g.d / 8), 64 * strip_waves<LC>(), 0, stream>>>(g, chunks);
    return hipGetLastError();
}

// More sketch columns than the accumulators of eight waves hold: sixteen waves to a strip, with accumulators for kSorsManyK, and the strip to as many
// work-groups as these need or as compute units are idle otherwise; each transforms all tokens for itself.  What bounds it: a chunk of 2048 tokens is
// 2.1 us of transform (n = 16384, next to no sketch columns) and 0.84 us for the 8192 rows gathered from LDS, 32 bytes at random places.  It
// takes the place of strips of four, two or one columns with all tokens in LDS, whose loads took 8, 4 or 2 bytes of a line (forward / backward
// 10938 x 560 -> 560, k = 5469: 83.5 / 118.1 -> 41.5 / 75.8 us; 14272 x 3072 -> 576, k = 12845: 362 / 223 -> 212 / 174; 58 such passes of
// up to 16384 tokens 0.36 to 0.92 of the time), and of chunks of 4096 (3236 x 528 -> 320, k = 2912: 18.0 / 31.0 -> 15.3 / 27.5).
// The column sums ride along as in the other strips; the first work-group of a strip writes them.
template <bool SUMS>
__global__ void __launch_bounds__(1024) sors_many_kernel(SorsArgs g, int chunks, int parts, int64_t part_k) {
    __shared__ float4 planes[StripShape<11>::REGION];
    __shared__ uint32_t sign_words[1024];
    sors_strip_body<11, true, 1, 16, SUMS, kSorsManyK / 4 / 1024>(g, chunks, planes, sign_words, blockIdx.x, gridDim.x, parts, part_k);
}
hipError_t launch_many(const SorsArgs &g, int chunks, hipStream_t stream) {
    const SorsParts p = sors_parts(g.d, g.k);
    const unsigned grid = (unsigned)(g.d / 8 * p.parts);
    if (g.colsum != nullptr)
        sors_many_kernel<true><<<grid, 1024, 0, stream>>>(g, chunks, (int)p.parts, p.part_k);
    else
        sors_many_kernel<false><<<grid, 1024, 0, stream>>>(g, chunks, (int)p.parts, p.part_k);
    return hipGetLastError();
}

}  // namespace

// (d: the 64 rows of a load stay inside one buffer descriptor, below the offset that stands for none)
bool sors_fast_ok(int64_t n, int64_t d) { return d % 8 == 0 && d < (1 << 22) && n >= 1 && n <= 32768; }

hipError_t launch_sors_bf16(const bf16_t *A, bf16_t *out, int64_t n, int64_t d, int64_t k, SketchState st,
                            hipStream_t stream, bf16_t *colsum, bool accumulate) {
    SorsArgs g{A, out, n, d, k, st, 1.0f / sqrtf((float)k), colsum, accumulate ? 1 : 0};
    // A kernel's transform length is at least 512; for fewer tokens the rows drawn below n_pad
    // are rows of the larger Walsh-Hadamard matrix restricted to its leading n_pad x n_pad block,
    // which is the n_pad-point matrix itself.
    const int l = sors_log(n);
    if (l > 15) return hipErrorInvalidValue;
    if (l >= 12) return k <= kSorsAccMaxK ? launch_strip<11, true>(g, sors_chunks(n), stream) : launch_many(g, sors_chunks(n), stream);  // chunks of 2048 tokens
    switch (l) {
        case 9: return launch_strip<9, false>(g, 1, stream);
        case 10: return launch_strip<10, false>(g, 1, stream);
        case 11: return launch_strip<11, false>(g, 1, stream);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_sors_colsum_bf16(const bf16_t *A, bf16_t *colsum, int64_t n, int64_t d, int64_t k, bool accumulate, hipStream_t stream) {
    const SorsArgs g{A, nullptr, n, d, k, SketchState{}, 0.0f, colsum, accumulate ? 1 : 0};
    const int l = sors_log(n);  // (chunks: see launch_sors_bf16)
    if (l >= 12) return launch_colsum_strips<11>(g, sors_chunks(n), stream);
    switch (l) {
        case 9: return launch_colsum_strips<9>(g, 1, stream);
        case 10: return launch_colsum_strips<10>(g, 1, stream);
        case 11: return launch_colsum_strips<11>(g, 1, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace rmm
