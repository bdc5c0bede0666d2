// Launchers of the streaming matrix-core schedule (packed and float32 input).
#include "launch.hpp"

namespace lce {
namespace {

template <int OUT, int MB, int NB>
void launch_vec(const StreamParams &p, dim3 grid, size_t lds, hipStream_t s) {
    const dim3 block(kMfmaThreads);
    if (p.region_vec == 0)
        hipLaunchKernelGGL((bconv2d_mfma_stream_kernel<OUT, MB, NB, 0>), grid, block, lds, s, p);
    else if (p.region_vec == 4)
        hipLaunchKernelGGL((bconv2d_mfma_stream_kernel<OUT, MB, NB, 4>), grid, block, lds, s, p);
    else if (p.region_vec == 2)
        hipLaunchKernelGGL((bconv2d_mfma_stream_kernel<OUT, MB, NB, 2>), grid, block, lds, s, p);
    else
        hipLaunchKernelGGL((bconv2d_mfma_stream_kernel<OUT, MB, NB, 1>), grid, block, lds, s, p);
}

template <int OUT>
void launch_out(const StreamParams &p, int mb, int nb, dim3 grid, size_t lds, hipStream_t s) {
    if (nb == 1)
        launch_vec<OUT, 4, 1>(p, grid, lds, s);
    else if (mb == 4)
        launch_vec<OUT, 4, 2>(p, grid, lds, s);
    else
        launch_vec<OUT, 2, 2>(p, grid, lds, s);
}

}  // namespace

void launch_mfma_stream(const StreamParams &p, int out_type, int mb, int nb, dim3 grid,
                        size_t lds, hipStream_t s) {
    switch (out_type) {
        case OUT_FLOAT: launch_out<OUT_FLOAT>(p, mb, nb, grid, lds, s); break;
        case OUT_BITS: launch_out<OUT_BITS>(p, mb, nb, grid, lds, s); break;
        default: launch_out<OUT_INT>(p, mb, nb, grid, lds, s); break;
    }
}

}  // namespace lce
