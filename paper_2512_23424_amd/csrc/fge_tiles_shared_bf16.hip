// 256x256 tile kernels, plain and gated, whose last tiles are shared between workgroups.
#include "fge_launch.h"
namespace fge {
template <> hipError_t launch_shared<bf16_t>(bool gated, int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a) {
    return launch_shared_any<bf16_t>(gated, out_dtype, grid, s, a);
}
}  // namespace fge
