// 256x256 tile kernels, plain and gated, whose last tiles are shared between workgroups.
#include "fge_launch.h"
namespace fge {
template <> hipError_t launch_shared<f8_t>(bool gated, int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a) {
    return launch_shared_any<f8_t>(gated, out_dtype, grid, s, a);
}
}  // namespace fge
