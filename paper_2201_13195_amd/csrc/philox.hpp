// Device-side Philox-4x32-10 and the counter -> sketch-entry map.
//
// The sketch S of the RMM layer (paper: Section 2.1, Eq. 5; Algorithm 1 "generate /
// rematerialize S") is never stored: every kernel that needs a piece of it calls
// these functions.  The element map is the one documented in include/rmm.h.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rmm {

struct SketchState {
    uint32_t key0, key1;  // seed lo / hi
    uint32_t off0, off1;  // offset lo / hi  (counter words 2 and 3)
    uint32_t row_mask;    // SORS kind only: n_pad - 1, n_pad = the token count rounded up to a power of two
};

// `n` = the sketch's token count; it enters the SORS kind only (through n_pad).
__host__ __device__ inline SketchState make_state(uint64_t seed, uint64_t offset, int64_t n = 1) {
    SketchState s;
    s.key0 = (uint32_t)seed;
    s.key1 = (uint32_t)(seed >> 32);
    s.off0 = (uint32_t)offset;
    s.off1 = (uint32_t)(offset >> 32);
    uint32_t n_pad = 1;
    while ((int64_t)n_pad < n && n_pad < 0x80000000u) n_pad <<= 1;
    s.row_mask = n_pad - 1u;
    return s;
}

// Counter word 1 (the slot of the sketch column) of the calls behind the SORS kind's token signs
// and selected rows; no sketch has that many columns.
constexpr uint32_t kSorsSignColumn = 0xFFFFFFFFu, kSorsRowColumn = 0xFFFFFFFEu;

struct Words4 {
    uint32_t w[4];
};

// One round of Philox-4x32.  The two 32x32->64 products map to v_mad_u64_u32 and each
// three-way xor to one v_bitop3_b32 (truth table 0x96 = a ^ b ^ c).
__device__ __forceinline__ void philox_round(uint32_t &c0, uint32_t &c1, uint32_t &c2, uint32_t &c3, uint32_t k0, uint32_t k1) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
    const uint32_t n0 = __builtin_amdgcn_bitop3_b32((uint32_t)(p1 >> 32), c1, k0, 0x96);
    const uint32_t n2 = __builtin_amdgcn_bitop3_b32((uint32_t)(p0 >> 32), c3, k1, 0x96);
    c1 = (uint32_t)p1;
    c3 = (uint32_t)p0;
    c0 = n0;
    c2 = n2;
}
constexpr uint32_t kPhiloxBump0 = 0x9E3779B9u, kPhiloxBump1 = 0xBB67AE85u;  // Weyl constants of the key

// One Philox-4x32-10 block: ten rounds, key bumped by the Weyl constants before rounds 2..10.
__device__ __forceinline__ Words4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                                uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) philox_round(c0, c1, c2, c3, k0 + (uint32_t)r * kPhiloxBump0, k1 + (uint32_t)r * kPhiloxBump1);
    Words4 o;
    o.w[0] = c0;
    o.w[1] = c1;
    o.w[2] = c2;
    o.w[3] = c3;
    return o;
}

// Box-Muller pair of one 32-bit word to fp32 precision (fp32 kernels).
// u1 = (hi16 + 1/2) / 2^16 in (0,1), u2 = lo16 / 2^16 in [0,1).
// Radius: v_log_f32 and v_sqrt_f32 (over all 2^16 arguments 0.39 ulp rms, 1.5 at most; sqrtf(-2 logf) 0.45 and 1.6).
// Angle: the distance t to the nearest quarter turn is exact, in quarter turns (a multiple of 2^-14 within
// +-1/2); its sine and cosine come from their Taylor series in t up to t^9 and t^10 (the next terms are below
// 2^-28), the sine's first coefficient in two parts (0.30 ulp rms, 0.89 at most; sincospif 0.31 and 0.93).
// Entries: 0.58 ulp rms, against 0.63 with the library functions (fp64 as the measure, 2^22 entries), at about
// half their instructions: the generator is what the fp32 sketch products wait for.
__device__ __forceinline__ void gauss_pair_precise(uint32_t w, float &z_cos, float &z_sin) {
    const float u1 = fmaf((float)(w >> 16), 1.0f / 65536.0f, 1.0f / 131072.0f);  // (exact)
    const float rad = __builtin_amdgcn_sqrtf(-1.3862943611198906f * __builtin_amdgcn_logf(u1));  // -2 ln2 log2 u1
    const float t = (float)((int)(w << 18) >> 18) * (1.0f / 16384.0f), tt = t * t;  // (the lowest 14 bits with their sign)
    const uint32_t quarter = w + 0x2000u;  // bits 14 and 15: its number
    float s = fmaf(tt, 1.6044118478735983e-4f, -4.681754135318688e-3f);  // (pi/2)^9 / 9!, -(pi/2)^7 / 7!
    s = fmaf(tt, s, 7.969262624616705e-2f);                              // (pi/2)^5 / 5!
    s = fmaf(tt, s, -6.459640975062463e-1f);                             // -(pi/2)^3 / 3!
    s = fmaf(t, 0x1.921fb6p+0f, t * fmaf(tt, s, -0x1.777a5cp-25f));      // pi/2 = 0x1.921fb6p+0 - 0x1.777a5cp-25
    float c = fmaf(tt, -2.5202042373060607e-5f, 9.192602748394266e-4f);  // -(pi/2)^10 / 10!, (pi/2)^8 / 8!
    c = fmaf(tt, c, -2.0863480763352960e-2f);                            // -(pi/2)^6 / 6!
    c = fmaf(tt, c, 2.5366950790104803e-1f);                             // (pi/2)^4 / 4!
    c = fmaf(tt, c, -1.2337005501361697f);                               // -(pi/2)^2 / 2!
    c = fmaf(tt, c, 1.0f);
    const bool odd = (quarter & 0x4000u) != 0;  // a quarter turn: (cos, sin) -> (-sin, cos)
    const float zc = odd ? s : c, zs = odd ? c : s;
    z_cos = rad * __uint_as_float(__float_as_uint(zc) ^ (((quarter + 0x4000u) << 16) & 0x80000000u));
    z_sin = rad * __uint_as_float(__float_as_uint(zs) ^ ((quarter << 16) & 0x80000000u));
}

// Unscaled sketch entry P[i][j] computed on its own (one Philox call per entry):
// the slow, obvious form used by the fp32 kernels and the debug export.
__device__ __forceinline__ float sketch_entry_precise(int kind, const SketchState &st, int64_t i, int64_t j) {
    if (kind == 0) {  // Gaussian
        const Words4 r = philox4x32_10((uint32_t)(i >> 3), (uint32_t)j, st.off0, st.off1, st.key0, st.key1);
        float zc, zs;
        gauss_pair_precise(r.w[(i & 7) >> 1], zc, zs);
        return (i & 1) ? zs : zc;
    }
    if (kind == 2) {  // SORS: sign of token i times entry (r_j, i) of the Walsh-Hadamard matrix
        const Words4 rs = philox4x32_10((uint32_t)(i >> 7), kSorsSignColumn, st.off0, st.off1, st.key0, st.key1);
        const Words4 rr = philox4x32_10((uint32_t)(j >> 2), kSorsRowColumn, st.off0, st.off1, st.key0, st.key1);
        const uint32_t t = (uint32_t)(i & 127);
        const uint32_t row = rr.w[j & 3] & st.row_mask;
        const uint32_t bit = ((rs.w[t >> 5] >> (t & 31)) ^ (uint32_t)__popc(row & (uint32_t)i)) & 1u;
        return bit ? -1.0f : 1.0f;
    }
    const Words4 r = philox4x32_10((uint32_t)(i >> 7), (uint32_t)j, st.off0, st.off1, st.key0, st.key1);
    const uint32_t t = (uint32_t)(i & 127);
    const uint32_t bit = (r.w[t >> 5] >> (t & 31)) & 1u;
    return bit ? -1.0f : 1.0f;
}

}  // namespace rmm
