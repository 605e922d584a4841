// Tile kernels for results of any width and row alignment.
#include "fge_launch.h"
namespace fge {
hipError_t launch_any_f8(int tile, int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a) {
    return launch_any_rows<f8_t, false>(tile, out_dtype, grid, s, a);
}
}  // namespace fge
