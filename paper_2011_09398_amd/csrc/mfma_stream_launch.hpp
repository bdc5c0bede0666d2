// Instances of the streaming schedule, for both filter layouts (two translation
// units, compiled in parallel).
#pragma once

#include "launch.hpp"

namespace lce {
namespace stream_launch {

template <int OUT, int MB, int NB, bool OHWI>
void launch_vec(const StreamParams &p, dim3 grid, size_t lds, hipStream_t s) {
    const dim3 block(kMfmaThreads);
    if (p.region_vec == 0) {
        if constexpr (!OHWI)
            hipLaunchKernelGGL((bconv2d_mfma_stream_kernel<OUT, MB, NB, 0>), grid, block, lds, s, p);
    } else if (p.region_vec == 4) {
        hipLaunchKernelGGL((bconv2d_mfma_stream_kernel<OUT, MB, NB, 4, OHWI>), grid, block, lds, s,
                           p);
    } else if (p.region_vec == 2) {
        hipLaunchKernelGGL((bconv2d_mfma_stream_kernel<OUT, MB, NB, 2, OHWI>), grid, block, lds, s,
                           p);
    } else {
        hipLaunchKernelGGL((bconv2d_mfma_stream_kernel<OUT, MB, NB, 1, OHWI>), grid, block, lds, s,
                           p);
    }
}

template <int OUT, bool OHWI>
void launch_out(const StreamParams &p, int mb, int nb, dim3 grid, size_t lds, hipStream_t s) {
    if (nb == 1)
        launch_vec<OUT, 4, 1, OHWI>(p, grid, lds, s);
    else if (mb == 4)
        launch_vec<OUT, 4, 2, OHWI>(p, grid, lds, s);
    else
        launch_vec<OUT, 2, 2, OHWI>(p, grid, lds, s);
}

template <bool OHWI>
void launch(const StreamParams &p, int out_type, int mb, int nb, dim3 grid, size_t lds,
            hipStream_t s) {
    switch (out_type) {
        case OUT_FLOAT: launch_out<OUT_FLOAT, OHWI>(p, mb, nb, grid, lds, s); break;
        case OUT_BITS: launch_out<OUT_BITS, OHWI>(p, mb, nb, grid, lds, s); break;
        default: launch_out<OUT_INT, OHWI>(p, mb, nb, grid, lds, s); break;
    }
}

}  // namespace stream_launch
}  // namespace lce
