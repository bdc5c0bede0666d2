// Launchers of the streaming matrix-core schedule on packed filters as they are
// stored (lce_bconv2d).
#include "mfma_stream_launch.hpp"

namespace lce {

void launch_mfma_stream_ohwi(const StreamParams &p, int out_type, int mb, int nb, dim3 grid,
                             size_t lds, hipStream_t s) {
    stream_launch::launch<true>(p, out_type, mb, nb, grid, lds, s);
}

}  // namespace lce
