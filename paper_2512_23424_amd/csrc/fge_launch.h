// Host-side table of tile configurations and the launchers each translation unit provides.
#pragma once
#include "fge_tile_kernel.h"

namespace fge {

enum TileId { TILE_64x64 = 0, TILE_64x512 = 1, TILE_128x128 = 2, TILE_256x256 = 3, TILE_PANEL = 4, TILE_64x128 = 5,
              TILE_GATED = 6, TILE_128x256 = 7, TILE_256x128 = 8, TILE_128x128_W8 = 9, TILE_128x128_S3 = 10, TILE_COUNT = 11 };

// coop_per_cu: workgroups of this tile's cooperative kernel that are resident on one CU at the
// same time (from the compiler's register / LDS report; a lower bound is safe), 0 if the tile
// has no cooperative kernel.
struct TileInfo { int bm, bn, threads, waves_n, coop_per_cu; const char *name, *name_split; };

inline const TileInfo &tile_info(int id) {
    static const TileInfo t[TILE_COUNT] = {
        {64, 64, 256, 2, 0, "64x64_w2x2", "64x64_w2x2_splitbf16"},
        {64, 512, 256, 4, 0, "64x512_w1x4", "64x512_w1x4_splitbf16"},
        {128, 128, 256, 2, 2, "128x128_w2x2", "128x128_w2x2_splitbf16"},
        {256, 256, 512, 4, 1, "256x256_w2x4", nullptr},
        // persistent narrow-K kernel, fp32 operands, always the split product
        {64, 512, 512, 8, 0, "panel64x512_w1x8_splitbf16", "panel64x512_w1x8_splitbf16"},
        {64, 128, 256, 2, 2, "64x128_w2x2", "64x128_w2x2_splitbf16"},
        // gated form, 16-bit operands: 256 rows x 128 output columns (two 256x128 products)
        {256, 128, 512, 4, 1, "gated256x128_w2x4", nullptr},
        // 16-bit and 8-bit operands: half a 256x256 tile either way, eight waves of 64x64 - twice the
        // workgroups of the 256x256 tiling for problems that leave it short of them
        {128, 256, 512, 4, 1, "128x256_w2x4", nullptr},
        {256, 128, 512, 2, 1, "256x128_w4x2", nullptr},
        // fp32 operands, split product: the 128x128 tile on eight waves of 64x32 (one workgroup per
        // CU) - for problems that give a CU one tile only, where the four-wave form leaves each
        // SIMD a single wave and nothing to run under its stalls
        {128, 128, 512, 4, 1, nullptr, "128x128_w2x4_splitbf16"},
        // 16- and 8-bit operands, at most one 128x128 tile per CU: eight waves of 64x32 and three
        // stage buffers (no second workgroup shares the CU, so a second K-tile copy in flight and a
        // second wave per SIMD hide the latencies instead); the plan puts it in the place of
        // 128x128_w2x2 wherever that tile is chosen for such a problem.  With a long K: four stage
        // buffers, the waves sharing out K, and two strips of 64 columns instead of four (tile_strips)
        {128, 128, 512, 4, 1, "128x128_w2x4_s3", nullptr},
    };
    return t[id];
}

// K from which the 64x64 and the 128x128_s3 tile run their K-sharing mainloop: 2 KB of K, the line where its
// slower start and end are paid for (6144 x 304 x 528 bf16: 9.4 us without, 10.2 with it; 2048 x 624 x 1544
// RMSNorm 16.5 / 17.3, 2048 x 1024 x 1544 18.4 / 18.0, 2048 x 2048 x 1544 26.1 / 24.3 us).
inline bool long_k(int K, size_t esize) { return (size_t)K * esize >= 2048; }
// K up to which the 256x256 tile and the gated form run the loop over k-steps: four K tiles of 64 16-bit values,
// one of 128 8-bit ones.  The quadrants' loop copies two K tiles before it multiplies the first, which a short K does
// not make up for (quadrants / k-steps, us; bf16 8192 x K x 4096, no row op: K = 64 24.9 / 24.0, 256 32.2 / 32.1, 384 38.6 / 39.5;
// RMSNorm in one kernel: 128 45.7 / 44.7, 256 51.0 / 51.5, 512 62.5 / 63.6; softmax in 16 problems of 2048 x K x 2048: 128 103.8 /
// 100.7, 256 115.4 / 114.8, 640 152.4 / 154.8; gated: 64 42.8 / 40.7, 256 62.6 / 60.9, 384 76.1 / 76.4, 640 98.4 / 102; E4M3: 128 23.3 / 22.5,
// 144 26.2 / 27.0, 256 26.2 / 25.8, 384 28.6 / 29.2, RMSNorm 256 45.4 / 45.6).
inline bool short_k(int K, size_t esize) { return (size_t)K * esize <= (esize == 2 ? 512 : 128); }
// Wave strips across a tile.  any_rows: the forms for results of any width, which share out K always.
inline int tile_strips(int tile, int K, size_t esize, bool any_rows) {
    return tile == TILE_128x128_S3 && (any_rows || long_k(K, esize)) ? 2 : tile_info(tile).waves_n;
}

// Defined in fge_tiles_f32.hip / fge_tiles_f32s.hip / fge_tiles_bf16.hip (separate units so they
// compile in parallel).  f32: fp32 matrix instruction; f32s: split-bf16 product.
hipError_t launch_tile_f32(int tile, int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a);
hipError_t launch_tile_f32s(int tile, int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a);
hipError_t launch_tile_bf16(int tile, int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a);
hipError_t launch_tile_f16(int tile, int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a);
hipError_t launch_tile_f8(int tile, int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a);
// Defined in fge_panel_f32.hip: the persistent narrow-K kernel (grid = number of workgroups).
hipError_t launch_panel_f32(int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a);

// Element-granular kernels (fge_generic.hip) for shapes the vectorised kernels do not take.
// gemm: dst = act(post*(alpha*X.W^T + b)); act: dst = act(X) [* W if W is set] with X (and W) laid
// out like dst; row:
// dst = rowop(X) with X rows x N at strides (ldx, bsx).  M rows per problem, `batch` problems.
struct GenArgs {
    const void *X, *W;
    const float *b, *gamma, *beta;
    const float *b2;            // slice sum with a gate: bias of the second product
    void *dst;
    float *aux;
    int M, N, K, batch;
    int64_t ldx, ldw, ldd, bsx, bsd;
    float alpha, post, lo, hi, eps;
    int act, norm;
};
hipError_t launch_generic_gemm(int in_dtype, int dst_dtype, hipStream_t s, const GenArgs &a);
hipError_t launch_generic_act(int dtype, hipStream_t s, const GenArgs &a);
hipError_t launch_generic_row(int src_dtype, int out_dtype, hipStream_t s, const GenArgs &a);
// X: a.K dense fp32 slices of M x N, a.bsx elements apart; dst = act(post*(alpha*sum + b)),
// times post*(alpha*sum2 + b2) when W points to the slices of a second product (gated form)
hipError_t launch_splitk_sum(int dst_dtype, hipStream_t s, const GenArgs &a);

// Dense, zero-padded copy of an operand (fge_generic.hip): dst is rows_dst x Kp of the same
// element type, Kp a multiple of the 16-byte chunk; source: batch problems of M rows x K.
struct PadArgs {
    const void *src;
    void *dst;
    int M, batch, K, Kp;
    int64_t ld, bs;             // source row stride / stride between problems, in elements
    int64_t rows_dst;           // >= batch * M; the rows beyond are zero
};
hipError_t launch_pad_rows(int dtype, hipStream_t s, const PadArgs &a);
hipError_t launch_pad_vec(const float *src, float *dst, int n, int np, hipStream_t s);

// Workgroups of `kernel` the current device holds at the same time (0 if the query fails).
inline int resident_workgroups(const void *kernel, int threads) {
    int per_cu = 0, dev = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess) return 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    return per_cu * cus;
}

// Which tiles exist for which operand type (tile selection on the host must agree):
//   bf16, fp16, fp8: 64x64, 64x512, 128x128 (+ cooperative; four waves, and eight with three
//         stage buffers for one tile per CU), 256x256 and its halves 128x256, 256x128 (+ cooperative)
//   fp32: 64x64, 64x512, 64x128 (+ cooperative) - once with the fp32 matrix instruction and once
//         with the split-bf16 product (SPLIT); 128x128 (+ cooperative; four waves, and eight for one
//         tile per CU) with the split product only
// The 16-bit output type that goes with an operand type (the other output type is fp32).
template <typename InT> struct NarrowOut { typedef bf16_t type; };
template <> struct NarrowOut<f16_t> { typedef f16_t type; };

// 256x256 tiles and the gated form over a short K; defined in fge_tiles_short_*.hip.
template <typename InT> hipError_t launch_short(bool gated, int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a);

// ... and with shared tiles (a.share; ordinary launches); defined in fge_tiles_shared_*.hip.
template <typename InT> hipError_t launch_shared(bool gated, int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a);

// The 256x256 tile, ordinary and cooperative launch: a kernel for every row op.  The four groups of a wave's rows
// each pass over the code of all row ops and activations, and where one kernel holds all of them (90 to 105 KB) its
// instructions arrive late, by an amount that any change of that code moves (bf16, ordinary: 8192 x 4096 x 4096 SiLU 212
// to 217 us, 8192 x 64 x 4096 27.5 to 30.4 us).
// STAGES: as for the tile kernel.  FULL (cooperative form): every tile lies inside the matrix, no guards.  All workgroups of
// a cooperative grid must be resident at once; one that the device cannot hold that way is refused.
template <typename InT, int STAGES, bool SHARED = false>
inline hipError_t launch_256(int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a) {
    typedef typename NarrowOut<InT>::type NarrowT;
#define FGE_256_KERNEL(OT, COOP, FULL, NORM)                                                    \
    do {                                                                                        \
        auto kern = tile_kernel<InT, OT, 256, 256, 2, 4, COOP, FULL, false, false, STAGES, false, NORM, SHARED>; \
        if (COOP) {                                                                             \
            static const int resident = resident_workgroups(reinterpret_cast<const void *>(kern), 512); \
            if ((int)grid.x > resident) return hipErrorCooperativeLaunchTooLarge;               \
        }                                                                                       \
        hipLaunchKernelGGL(kern, grid, dim3(512), 0, s, a);                                     \
    } while (0)
#define FGE_256(COOP, FULL, NORM)                                                               \
    do {                                                                                        \
        if (out_dtype != FGE_F32) FGE_256_KERNEL(NarrowT, COOP, FULL, NORM);                    \
        else                      FGE_256_KERNEL(float, COOP, FULL, NORM);                      \
    } while (0)
#define FGE_256_FORM(NORM)                                                                      \
    do {                                                                                        \
        if constexpr (SHARED)                       FGE_256(false, false, NORM);                \
        else if (!a.coop)                           FGE_256(false, false, NORM);                \
        else if (a.M % 256 == 0 && a.N % 256 == 0)  FGE_256(true, true, NORM);                  \
        else                                        FGE_256(true, false, NORM);                 \
    } while (0)
    switch (a.norm) {
    case FGE_NORM_NONE:      FGE_256(false, false, FGE_NORM_NONE); break;
    case FGE_NORM_SOFTMAX:   FGE_256_FORM(FGE_NORM_SOFTMAX); break;
    case FGE_NORM_LAYERNORM: FGE_256_FORM(FGE_NORM_LAYERNORM); break;
    case FGE_NORM_RMSNORM:   FGE_256_FORM(FGE_NORM_RMSNORM); break;
    default:                 FGE_256_FORM(FGE_NORM_LOGSUMEXP); break;
    }
#undef FGE_256_FORM
#undef FGE_256
#undef FGE_256_KERNEL
    return hipGetLastError();
}

template <typename InT, bool SPLIT>
inline hipError_t launch_tile_any(int tile, int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a) {
    typedef typename NarrowOut<InT>::type NarrowT;
#define FGE_LAUNCH(BM, BN, WM, WN)                                                              \
    do {                                                                                        \
        if (out_dtype != FGE_F32)                                                               \
            hipLaunchKernelGGL((tile_kernel<InT, NarrowT, BM, BN, WM, WN, false, false, SPLIT>), grid, \
                               dim3(64 * WM * WN), 0, s, a);                                    \
        else                                                                                    \
            hipLaunchKernelGGL((tile_kernel<InT, float, BM, BN, WM, WN, false, false, SPLIT>), grid, \
                               dim3(64 * WM * WN), 0, s, a);                                    \
    } while (0)
    // cooperative kernel of a tile.  All workgroups of the grid must be resident at once; a
    // launch that the device cannot hold that way is refused instead of being left to run into
    // its wait limit.
#define FGE_LAUNCH_COOP1(BM, BN, WM, WN, OT, NORM)                                              \
    do {                                                                                        \
        auto kern = tile_kernel<InT, OT, BM, BN, WM, WN, true, false, SPLIT, false, 0, false, NORM>; \
        static const int resident = resident_workgroups(reinterpret_cast<const void *>(kern), 64 * WM * WN); \
        if ((int)grid.x > resident) return hipErrorCooperativeLaunchTooLarge;                   \
        hipLaunchKernelGGL(kern, grid, dim3(64 * WM * WN), 0, s, a);                            \
    } while (0)
#define FGE_LAUNCH_COOP(BM, BN, WM, WN, NORM)                                                   \
    do {                                                                                        \
        if (out_dtype != FGE_F32)  FGE_LAUNCH_COOP1(BM, BN, WM, WN, NarrowT, NORM);             \
        else                       FGE_LAUNCH_COOP1(BM, BN, WM, WN, float, NORM);               \
    } while (0)
    // 128x128 tiles on eight waves with more stage buffers (one workgroup per CU), ordinary and cooperative launch
#define FGE_LAUNCH_DEEP128(OT, WM, WN, STAGES)                                                  \
    do {                                                                                        \
        if (a.coop) {                                                                           \
            auto kern = tile_kernel<InT, OT, 128, 128, WM, WN, true, false, false, false, STAGES>; \
            static const int resident = resident_workgroups(reinterpret_cast<const void *>(kern), 512); \
            if ((int)grid.x > resident) return hipErrorCooperativeLaunchTooLarge;               \
            hipLaunchKernelGGL(kern, grid, dim3(512), 0, s, a);                                 \
        } else {                                                                                \
            hipLaunchKernelGGL((tile_kernel<InT, OT, 128, 128, WM, WN, false, false, false, false, STAGES>), grid, \
                               dim3(512), 0, s, a);                                             \
        }                                                                                       \
    } while (0)
    const bool long_row = long_k(a.K, sizeof(InT));
    constexpr bool BF = sizeof(InT) <= 2;
    switch (tile) {
    case TILE_64x64:
        if constexpr (BF) {
            if (long_row) {
                if (out_dtype != FGE_F32)
                    hipLaunchKernelGGL((tile_kernel<InT, NarrowT, 64, 64, 2, 2, false, false, false, false, 4>), grid, dim3(256), 0, s, a);
                else
                    hipLaunchKernelGGL((tile_kernel<InT, float, 64, 64, 2, 2, false, false, false, false, 4>), grid, dim3(256), 0, s, a);
                break;
            }
        }
        FGE_LAUNCH(64, 64, 2, 2);
        break;
    case TILE_64x512:  FGE_LAUNCH(64, 512, 1, 4); break;
    case TILE_128x128:
        if constexpr (BF || SPLIT) {
            // (a cooperative kernel for every row op, as for the 256x256 tile: fp32 16669 x 32 x 256 softmax 16.8 us
            // with one for all)
            if (!a.coop)                           FGE_LAUNCH(128, 128, 2, 2);
            else if (a.norm == FGE_NORM_SOFTMAX)   FGE_LAUNCH_COOP(128, 128, 2, 2, FGE_NORM_SOFTMAX);
            else if (a.norm == FGE_NORM_LAYERNORM) FGE_LAUNCH_COOP(128, 128, 2, 2, FGE_NORM_LAYERNORM);
            else if (a.norm == FGE_NORM_RMSNORM)   FGE_LAUNCH_COOP(128, 128, 2, 2, FGE_NORM_RMSNORM);
            else                                   FGE_LAUNCH_COOP(128, 128, 2, 2, FGE_NORM_LOGSUMEXP);
            break;
        }
        return hipErrorInvalidValue;
    case TILE_128x128_S3:
        if constexpr (BF && !SPLIT) {
            if (out_dtype != FGE_F32) { if (long_row) FGE_LAUNCH_DEEP128(NarrowT, 4, 2, 4); else FGE_LAUNCH_DEEP128(NarrowT, 2, 4, 3); }
            else                      { if (long_row) FGE_LAUNCH_DEEP128(float, 4, 2, 4);   else FGE_LAUNCH_DEEP128(float, 2, 4, 3); }
            break;
        }
        return hipErrorInvalidValue;
    case TILE_256x256:
        if constexpr (BF) {
            if (short_k(a.K, sizeof(InT))) return launch_short<InT>(false, out_dtype, grid, s, a);
            if (a.share) return launch_shared<InT>(false, out_dtype, grid, s, a);
            return launch_256<InT, 0>(out_dtype, grid, s, a);
        }
        return hipErrorInvalidValue;
    case TILE_128x128_W8:
        if constexpr (SPLIT) {
            if (a.coop) FGE_LAUNCH_COOP(128, 128, 2, 4, -1);
            else        FGE_LAUNCH(128, 128, 2, 4);
            break;
        }
        return hipErrorInvalidValue;
    case TILE_64x128:
        if constexpr (!BF) {
            if (a.coop) FGE_LAUNCH_COOP(64, 128, 2, 2, -1);
            else        FGE_LAUNCH(64, 128, 2, 2);
            break;
        }
        return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
    }
#undef FGE_LAUNCH
#undef FGE_LAUNCH_DEEP128
#undef FGE_LAUNCH_COOP
#undef FGE_LAUNCH_COOP1
    return hipGetLastError();
}

// The gated tile kernel (16-bit and 8-bit operands), ordinary and cooperative launch: a kernel for every row op, as
// for the plain 256x256 tile (bf16 8192 x 384 x 4096 SiLU RMSNorm 106.9 us with one for all, 101.0 so; at K = 4096 439.8 and 432.4).
template <typename InT, int STAGES, bool SHARED = false>
inline hipError_t launch_gated_form(int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a) {
    typedef typename NarrowOut<InT>::type NarrowT;
#define FGE_GATED_KERNEL(OT, COOP, NORM)                                                        \
    do {                                                                                        \
        auto kern = tile_kernel<InT, OT, 256, 256, 2, 4, COOP, false, false, true, STAGES, false, NORM, SHARED>; \
        if (COOP) {                                                                             \
            static const int resident = resident_workgroups(reinterpret_cast<const void *>(kern), 512); \
            if ((int)grid.x > resident) return hipErrorCooperativeLaunchTooLarge;               \
        }                                                                                       \
        hipLaunchKernelGGL(kern, grid, dim3(512), 0, s, a);                                     \
    } while (0)
#define FGE_GATED(COOP, NORM)                                                                   \
    do {                                                                                        \
        if (out_dtype != FGE_F32) FGE_GATED_KERNEL(NarrowT, COOP, NORM);                        \
        else                      FGE_GATED_KERNEL(float, COOP, NORM);                          \
    } while (0)
#define FGE_GATED_FORM(NORM)                                                                    \
    do {                                                                                        \
        if constexpr (SHARED)  FGE_GATED(false, NORM);                                          \
        else if (a.coop)       FGE_GATED(true, NORM);                                           \
        else                   FGE_GATED(false, NORM);                                          \
    } while (0)
    switch (a.norm) {
    case FGE_NORM_NONE:      FGE_GATED(false, FGE_NORM_NONE); break;
    case FGE_NORM_SOFTMAX:   FGE_GATED_FORM(FGE_NORM_SOFTMAX); break;
    case FGE_NORM_LAYERNORM: FGE_GATED_FORM(FGE_NORM_LAYERNORM); break;
    case FGE_NORM_RMSNORM:   FGE_GATED_FORM(FGE_NORM_RMSNORM); break;
    default:                 FGE_GATED_FORM(FGE_NORM_LOGSUMEXP); break;
    }
#undef FGE_GATED_FORM
#undef FGE_GATED
#undef FGE_GATED_KERNEL
    return hipGetLastError();
}
template <typename InT>
inline hipError_t launch_gated_any(int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a) {
    if (a.share) return launch_shared<InT>(true, out_dtype, grid, s, a);
    return short_k(a.K, sizeof(InT)) ? launch_short<InT>(true, out_dtype, grid, s, a) : launch_gated_form<InT, 0>(out_dtype, grid, s, a);
}
// ... and the 256x256 tile, plain and gated, over a short K.
template <typename InT>
inline hipError_t launch_short_any(bool gated, int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a) {
    return gated ? launch_gated_form<InT, 2>(out_dtype, grid, s, a) : launch_256<InT, 2>(out_dtype, grid, s, a);
}
// ... and with shared tiles, in ordinary launches only: the tiles, then the sums of the shared ones.  (A launch of the cooperative gated form with shared tiles has
// faulted, cause not found: 2048 x 6888 x 4272 bf16 RMSNorm, one whole round and 34 tiles in four slices.  No cooperative
// kernel shares tiles, the plain ones included, which had the same code.)
template <typename InT>
inline hipError_t launch_shared_any(bool gated, int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a) {
    if (a.coop) return hipErrorInvalidValue;
    const hipError_t e = gated ? launch_gated_form<InT, 0, true>(out_dtype, grid, s, a) : launch_256<InT, 0, true>(out_dtype, grid, s, a);
    if (e != hipSuccess) return e;
    typedef typename NarrowOut<InT>::type NarrowT;
    const dim3 quarters((grid.x - (unsigned)a.share_from) / (unsigned)a.share * 4);
#define FGE_SHARED_FINISH(NORM)                                                                                     \
    do {                                                                                                            \
        if (out_dtype != FGE_F32) {                                                                                 \
            if (gated) hipLaunchKernelGGL((shared_finish_kernel<NarrowT, true, NORM>), quarters, dim3(512), 0, s, a);  \
            else       hipLaunchKernelGGL((shared_finish_kernel<NarrowT, false, NORM>), quarters, dim3(512), 0, s, a); \
        } else {                                                                                                    \
            if (gated) hipLaunchKernelGGL((shared_finish_kernel<float, true, NORM>), quarters, dim3(512), 0, s, a);    \
            else       hipLaunchKernelGGL((shared_finish_kernel<float, false, NORM>), quarters, dim3(512), 0, s, a);   \
        }                                                                                                           \
    } while (0)
    switch (a.norm) {
    case FGE_NORM_NONE:      FGE_SHARED_FINISH(FGE_NORM_NONE); break;
    case FGE_NORM_SOFTMAX:   FGE_SHARED_FINISH(FGE_NORM_SOFTMAX); break;
    case FGE_NORM_LAYERNORM: FGE_SHARED_FINISH(FGE_NORM_LAYERNORM); break;
    case FGE_NORM_RMSNORM:   FGE_SHARED_FINISH(FGE_NORM_RMSNORM); break;
    default:                 FGE_SHARED_FINISH(FGE_NORM_LOGSUMEXP); break;
    }
#undef FGE_SHARED_FINISH
    return hipGetLastError();
}
// The half-tile configurations (TILE_128x256, TILE_256x128), ordinary or cooperative launch;
// defined in fge_tiles_half.hip.
template <typename InT>
inline hipError_t launch_half_any(int tile, int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a) {
    typedef typename NarrowOut<InT>::type NarrowT;
#define FGE_HALF(BM, BN, WM, WN, OT)                                                            \
    do {                                                                                        \
        if (a.coop) {                                                                           \
            auto kern = tile_kernel<InT, OT, BM, BN, WM, WN, true, false>;                      \
            static const int resident = resident_workgroups(reinterpret_cast<const void *>(kern), 512); \
            if ((int)grid.x > resident) return hipErrorCooperativeLaunchTooLarge;               \
            hipLaunchKernelGGL(kern, grid, dim3(512), 0, s, a);                                 \
        } else {                                                                                \
            hipLaunchKernelGGL((tile_kernel<InT, OT, BM, BN, WM, WN, false, false>), grid, dim3(512), 0, s, a); \
        }                                                                                       \
    } while (0)
    if (tile == TILE_128x256) {
        if (out_dtype != FGE_F32) FGE_HALF(128, 256, 2, 4, NarrowT); else FGE_HALF(128, 256, 2, 4, float);
    } else if (tile == TILE_256x128) {
        if (out_dtype != FGE_F32) FGE_HALF(256, 128, 4, 2, NarrowT); else FGE_HALF(256, 128, 4, 2, float);
    } else {
        return hipErrorInvalidValue;
    }
#undef FGE_HALF
    return hipGetLastError();
}
// Results of any width and row alignment (ANY): ordinary launches of the tiles any_tile() leaves; defined in
// fge_tiles_any_*.hip.
template <typename InT, bool SPLIT>
inline hipError_t launch_any_rows(int tile, int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a) {
    typedef typename NarrowOut<InT>::type NarrowT;
    constexpr bool BF = sizeof(InT) <= 2;
#define FGE_ANY(BM, BN, WM, WN, STAGES)                                                                                \
    do {                                                                                                               \
        if (out_dtype != FGE_F32)                                                                                      \
            hipLaunchKernelGGL((tile_kernel<InT, NarrowT, BM, BN, WM, WN, false, false, SPLIT, false, STAGES, true>),  \
                               grid, dim3(64 * WM * WN), 0, s, a);                                                     \
        else                                                                                                           \
            hipLaunchKernelGGL((tile_kernel<InT, float, BM, BN, WM, WN, false, false, SPLIT, false, STAGES, true>),    \
                               grid, dim3(64 * WM * WN), 0, s, a);                                                     \
    } while (0)
    if (tile == TILE_64x64) FGE_ANY(64, 64, 2, 2, (BF ? 4 : 0));
    else if (tile == TILE_128x128 && (BF || SPLIT)) { if constexpr (BF || SPLIT) FGE_ANY(128, 128, 2, 2, 0); }
    else if (tile == TILE_128x128_W8 && SPLIT)      { if constexpr (SPLIT) FGE_ANY(128, 128, 2, 4, 0); }
    else if (tile == TILE_128x128_S3 && BF)         { if constexpr (BF) FGE_ANY(128, 128, 4, 2, 4); }
    else if (tile == TILE_256x256 && BF)            { if constexpr (BF) FGE_ANY(256, 256, 2, 4, 0); }
    else return hipErrorInvalidValue;
#undef FGE_ANY
    return hipGetLastError();
}
hipError_t launch_any_f32(int tile, int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a);
hipError_t launch_any_f32s(int tile, int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a);
hipError_t launch_any_bf16(int tile, int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a);
hipError_t launch_any_f16(int tile, int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a);
hipError_t launch_any_f8(int tile, int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a);
// The tile that stands in for one that has no kernel of that form.
inline int any_tile(int tile, int in_dtype, bool ieee_fp32) {
    const bool small_only = in_dtype == FGE_F32 && ieee_fp32;
    switch (tile) {
    case TILE_128x256: case TILE_256x128:          return TILE_256x256;
    case TILE_PANEL:                               return TILE_128x128;
    case TILE_64x512: case TILE_64x128:            return small_only ? TILE_64x64 : TILE_128x128;
    default:                                       return tile;
    }
}

hipError_t launch_half_bf16(int tile, int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a);
hipError_t launch_half_f16(int tile, int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a);
hipError_t launch_half_f8(int tile, int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a);
hipError_t launch_gated_bf16(int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a);
hipError_t launch_gated_f16(int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a);
hipError_t launch_gated_f8(int out_dtype, dim3 grid, hipStream_t s, const TileArgs &a);

// Defined in fge_skinny.hip: products of at most 64 rows (16- and 8-bit operands), and the row
// operation behind one as a kernel of its own.  cus: compute units of the device.
struct SkinnyArgs;
hipError_t launch_skinny(int in_dtype, bool gated, int cus, hipStream_t s, const SkinnyArgs &a);
hipError_t launch_skinny_rows(int in_dtype, bool gated, int cus, hipStream_t s, const SkinnyArgs &a);

// Whether launch_tile_any has a cooperative kernel for this tile and operand type.
inline bool tile_has_coop(int tile, int in_dtype) {
    if (tile == TILE_GATED) return true;
    if (tile == TILE_128x256 || tile == TILE_256x128) return in_dtype != FGE_F32;
    return in_dtype != FGE_F32 ? (tile == TILE_128x128 || tile == TILE_128x128_S3 || tile == TILE_256x256)
                               : (tile == TILE_64x128 || tile == TILE_128x128 || tile == TILE_128x128_W8);
}

}  // namespace fge
