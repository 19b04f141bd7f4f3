// Launcher of plain_pass_kernel, shared by the translation units that hold its instantiations
// (plain_pass_*.hip; separate files only to keep the build parallel).
#pragma once
#include "plain_kernels.hpp"

namespace rmm {

// Which tile shapes a launch uses.
struct PlainLaunch {
    PlainArgs ga, gs;
    ColsumArgs gc;
    int plain_blocks, sketch_blocks, colsum_blocks;
    int cfg;            // tile shape of the plain product
    int tile;           // the one of mfma_kernels.hpp in its place (launch_forward_pass_bf16x8), -1: none
    bool sketch_small;  // the 32 x 32 tile for the sketch product (never with PLAIN_BIG)
};

// One for each element type and way of loading it (plain_kernels.hpp: MODE 4, 3, 0); bf16: of A, then of W.
hipError_t launch_plain_pass_f32x4(const PlainLaunch &p, bool b_rows_k, hipStream_t stream);
hipError_t launch_plain_pass_f32(const PlainLaunch &p, bool b_rows_k, hipStream_t stream);
hipError_t launch_plain_pass_bf16(const PlainLaunch &p, bool b_rows_k, hipStream_t stream);  // 3, 3
hipError_t launch_forward_pass_bf16x8(const PlainLaunch &p, hipStream_t stream);             // 4, 4
hipError_t launch_backward_pass_bf16_x8(const PlainLaunch &p, hipStream_t stream);           // 3, 4
hipError_t launch_backward_pass_bf16x8_(const PlainLaunch &p, hipStream_t stream);           // 4, 3
hipError_t launch_plain_pass_far_f32(const PlainLaunch &p, bool b_rows_k, hipStream_t stream);   // PLAIN_TINY only
hipError_t launch_plain_pass_far_bf16(const PlainLaunch &p, bool b_rows_k, hipStream_t stream);  // PLAIN_TINY only

template <typename T, int MODE, int MODE_B, int BMODE, int SKETCH>
hipError_t launch_plain_pass_kind(const PlainLaunch &p, hipStream_t stream) {
    const unsigned grid = (unsigned)(p.plain_blocks + p.sketch_blocks + p.colsum_blocks);
#define RMM_PLAIN_PASS(S, SS)                                                                                        \
    plain_pass_kernel<T, S, SS, SKETCH, BMODE, MODE, MODE_B>                                                                \
        <<<grid, kPlainThreads, 0, stream>>>(p.ga, p.gs, p.gc, p.plain_blocks, p.sketch_blocks, p.colsum_blocks)
    if constexpr (MODE == 0) {
        RMM_PLAIN_PASS(PlainTiny, PlainTiny);
    } else {
        if (p.cfg == PLAIN_TINY) {
            bool small = p.sketch_small || p.sketch_blocks == 0;
            if constexpr (sizeof(T) == 4) small = true;  // (no slices)
            if (small)
                RMM_PLAIN_PASS(PlainTiny, PlainTiny);
            else
                RMM_PLAIN_PASS(PlainTiny, PlainSketch);
        } else if (p.cfg == PLAIN_BIG) {
            if constexpr (sizeof(T) == 2 && MODE == 4 && MODE_B == 4 && BMODE == PB_K)
                return hipErrorInvalidValue;  // (any_width_tile has others for it)
            else
                RMM_PLAIN_PASS(PlainBig, PlainSketch);
        } else if (p.sketch_small)
            RMM_PLAIN_PASS(PlainMid, PlainTiny);
        else
            RMM_PLAIN_PASS(PlainMid, PlainSketch);
    }
#undef RMM_PLAIN_PASS
    return hipGetLastError();
}

template <typename T, int MODE, int MODE_B, int BMODE>
hipError_t launch_plain_pass_rows(const PlainLaunch &p, hipStream_t stream) {
    return p.gs.kind == 0 ? launch_plain_pass_kind<T, MODE, MODE_B, BMODE, PA_GAUSS>(p, stream)
                          : launch_plain_pass_kind<T, MODE, MODE_B, BMODE, PA_SIGN>(p, stream);
}

template <typename T, int MODE>
hipError_t launch_plain_pass_impl(const PlainLaunch &p, bool b_rows_k, hipStream_t stream) {
    return b_rows_k ? launch_plain_pass_rows<T, MODE, MODE, PB_N>(p, stream) : launch_plain_pass_rows<T, MODE, MODE, PB_K>(p, stream);
}

}  // namespace rmm
