// Tile kernels for results of any width and row alignment.
#include "fge_launch.h"
namespace fge {
hipError_t launch_any_f32s(int tile, int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a) {
    return launch_any_rows<float, true>(tile, out_dtype, grid, s, a);
}
}  // namespace fge
