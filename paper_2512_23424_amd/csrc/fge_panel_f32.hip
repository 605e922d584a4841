// Instantiations of the persistent narrow-K kernel (fp32 operands, split-bf16 MFMA).
#include "fge_launch.h"
#include "fge_panel_kernel.h"
namespace fge {
namespace {
constexpr size_t LLC_BYTES = (size_t)256 << 20;     // memory-side cache in front of HBM

template <typename OutT, typename Shape>
void launch(dim3 grid, hipStream_t s, TileArgs a) {
    const bool full = a.M % Shape::BM == 0 && a.N == Shape::BN;
    const unsigned tiles = (unsigned)((a.M + Shape::BM - 1) / Shape::BM);
    if (grid.x > tiles) grid.x = tiles;
    // (rows that do not end on whole 64-byte sectors are not streamed: 400000 x 44 x 252 200.8 us so, 146.1 in 128x128 tiles;
    // 400000 x 44 x 256 streamed 83.6)
    const bool sectors = a.N * sizeof(OutT) % 64 == 0 && a.ldo * (int64_t)sizeof(OutT) % 64 == 0;
    const bool stream = (size_t)a.M * a.N * sizeof(OutT) >= LLC_BYTES && sectors;
    if (!sectors) a.stream_out = 0;
    const dim3 block(Shape::THREADS);
    // the chain this kernel exists for - clamp to a narrow range, then the row logsumexp - with
    // activation and row op fixed at compile time (fp32 results, tiles inside the matrix)
    if constexpr (sizeof(OutT) == 4 && Shape::WAVES_N == 8) {
        if (full && a.act == FGE_ACT_CLAMP && a.norm == FGE_NORM_LOGSUMEXP && a.hi - a.lo <= 64.0f) {
            if (stream) hipLaunchKernelGGL((panel_kernel<Shape, OutT, true, true, FGE_ACT_CLAMP, FGE_NORM_LOGSUMEXP, true>), grid, block, 0, s, a);
            else        hipLaunchKernelGGL((panel_kernel<Shape, OutT, true, false, FGE_ACT_CLAMP, FGE_NORM_LOGSUMEXP, true>), grid, block, 0, s, a);
            return;
        }
    }
    // else a kernel for every row op: one that holds the code of all of them spills registers (131072 x 32 x 364 SiLU
    // logsumexp 77.9 to 80.3 us, now 66.9; 65536 x 64 x 384 softmax 42.6 to 44.3)
#define FGE_PANEL(NORM)                                                                                                  \
    do {                                                                                                                 \
        if (full && stream) hipLaunchKernelGGL((panel_kernel<Shape, OutT, true, true, -1, NORM>), grid, block, 0, s, a);        \
        else if (full)      hipLaunchKernelGGL((panel_kernel<Shape, OutT, true, false, -1, NORM>), grid, block, 0, s, a);       \
        else if (stream)    hipLaunchKernelGGL((panel_kernel<Shape, OutT, false, true, -1, NORM>), grid, block, 0, s, a);       \
        else                hipLaunchKernelGGL((panel_kernel<Shape, OutT, false, false, -1, NORM>), grid, block, 0, s, a);      \
    } while (0)
    switch (a.norm) {
    case FGE_NORM_NONE:      FGE_PANEL(FGE_NORM_NONE); break;
    case FGE_NORM_SOFTMAX:   FGE_PANEL(FGE_NORM_SOFTMAX); break;
    case FGE_NORM_LAYERNORM: FGE_PANEL(FGE_NORM_LAYERNORM); break;
    case FGE_NORM_RMSNORM:   FGE_PANEL(FGE_NORM_RMSNORM); break;
    default:                 FGE_PANEL(FGE_NORM_LOGSUMEXP); break;
    }
#undef FGE_PANEL
}
}  // namespace

hipError_t launch_panel_f32(int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a) {
#define FGE_WIDTH(WN)                                                                   \
    do {                                                                                \
        if (out_dtype == FGE_BF16) launch<bf16_t, PanelShape<WN>>(grid, s, a);          \
        else                       launch<float, PanelShape<WN>>(grid, s, a);           \
    } while (0)
    if (a.N > 256)      FGE_WIDTH(8);
    else if (a.N > 128) FGE_WIDTH(4);
    else                FGE_WIDTH(2);
#undef FGE_WIDTH
    return hipGetLastError();
}
}  // namespace fge
