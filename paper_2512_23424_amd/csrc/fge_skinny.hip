// Launches of the few-row kernels (fge_skinny.h).
#include "fge_launch.h"
#include "fge_skinny.h"

namespace fge {

namespace {

// Ring depth: with at most one workgroup per CU the ring is as deep as LDS allows; with more of them
// several share a CU and cover each other.
template <typename InT, int MB, int CB, bool GATED> hipError_t launch_blocks(bool deep, dim3 grid, hipStream_t s, const SkinnyArgs &a) {
    constexpr int SUM = MB + CB;                      // 2 KB each per wave and K tile
    constexpr int DEEP = SUM <= 2 ? 4 : SUM == 3 ? 3 : SUM <= 5 ? 2 : 1, SHALLOW = SUM <= 2 ? 2 : 1;
    if (deep) hipLaunchKernelGGL((skinny_kernel<InT, MB, CB, GATED, DEEP>), grid, dim3(64 * SKINNY_WAVES), 0, s, a);
    else      hipLaunchKernelGGL((skinny_kernel<InT, MB, CB, GATED, SHALLOW>), grid, dim3(64 * SKINNY_WAVES), 0, s, a);
    return hipGetLastError();
}

// Blocks of 16 columns per workgroup.  One, as long as that gives a CU one workgroup at most; else two,
// for half the reads of X (16 x 4096 x 32000 56.7 -> 51.0 us, 64 x 4096 x 11008 35.2 -> 33.3 us) - but not where two
// leave a small second round of few-row workgroups (16 x 4096 x 11008: 22.8 against 20.6 us).
int column_blocks(bool gated, int M, int N, int cus) {
    const int g16 = (N + 15) / 16, g32 = (N + 31) / 32;
    if (gated || g16 <= cus) return 1;
    return M <= 16 && g32 > cus && g32 < 2 * cus ? 1 : 2;
}

template <typename InT, int MB> hipError_t launch_columns(bool gated, int cus, hipStream_t s, const SkinnyArgs &a) {
    const int cb = column_blocks(gated, a.M, a.N, cus);
    const int g = (a.N + 16 * cb - 1) / (16 * cb);
    const bool deep = g <= cus;
    if (gated)   return launch_blocks<InT, MB, 2, true>(deep, dim3(g), s, a);
    if (cb == 2) return launch_blocks<InT, MB, 2, false>(deep, dim3(g), s, a);
    return launch_blocks<InT, MB, 1, false>(deep, dim3(g), s, a);
}

template <typename InT> hipError_t launch_rows(bool gated, int cus, hipStream_t s, const SkinnyArgs &a) {
    if (a.M <= 16) return launch_columns<InT, 1>(gated, cus, s, a);
    if (a.M <= 32) return launch_columns<InT, 2>(gated, cus, s, a);
    return launch_columns<InT, 4>(gated, cus, s, a);
}

}  // namespace

hipError_t launch_skinny(int in_dtype, bool gated, int cus, hipStream_t s, const SkinnyArgs &a) {
    return in_dtype == FGE_BF16  ? launch_rows<bf16_t>(gated, cus, s, a)
           : in_dtype == FGE_F16 ? launch_rows<f16_t>(gated, cus, s, a)
                                 : launch_rows<f8_t>(gated, cus, s, a);
}

hipError_t launch_skinny_rows(int in_dtype, bool gated, int cus, hipStream_t s, const SkinnyArgs &a) {
    const dim3 grid((unsigned)a.M);
    const int cols = 16 * column_blocks(gated, a.M, a.N, cus), groups = (a.N + cols - 1) / cols;
#define FGE_ROWS(OT)                                                                                                        \
    do {                                                                                                                    \
        if (a.norm == FGE_NORM_LOGSUMEXP || a.N <= SKINNY_ROW_N)                                                            \
            hipLaunchKernelGGL((skinny_rows_kernel<OT, 64 * SKINNY_WAVES>), grid, dim3(64 * SKINNY_WAVES), 0, s, a, groups); \
        else                                                                                                                \
            hipLaunchKernelGGL((skinny_rows_kernel<OT, SKINNY_WIDE_NT>), grid, dim3(SKINNY_WIDE_NT), 0, s, a, groups);       \
    } while (0)
    if (in_dtype == FGE_F16) FGE_ROWS(f16_t);
    else                     FGE_ROWS(bf16_t);
#undef FGE_ROWS
    return hipGetLastError();
}

}  // namespace fge
