// Launchers of the streaming matrix-core schedule: packed and float32 input,
// filters in the layout of lce_bconv2d_mfma_weights.
#include "mfma_stream_launch.hpp"

namespace lce {

void launch_mfma_stream(const StreamParams &p, int out_type, int mb, int nb, dim3 grid,
                        size_t lds, hipStream_t s) {
    stream_launch::launch<false>(p, out_type, mb, nb, grid, lds, s);
}

}  // namespace lce
