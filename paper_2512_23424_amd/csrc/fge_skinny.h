// Products of few rows (at most 64, 16-bit and 8-bit operands): the weights are streamed once, every
// workgroup forms whole sums.
//
// Such a call reads N*K weights for M*N results: it is bound by how fast W arrives, and at these
// sizes (2 to 130 MB) by how much of it is in flight, not by arithmetic.  The tile kernels cut K
// into slices over workgroups to fill the chip and need fp32 partial products through memory and a
// second kernel that adds them; here a workgroup takes 16 (or 32) columns and ALL of K, so nothing but finished
// values leaves it:
//   * its eight waves share out the 128-byte K tiles of those columns (wave w: tiles w, w+8, ...,
//     so that the workgroup reads 1 KB runs of every row of W).  A wave copies its tiles of W and X
//     global -> LDS into a ring of its own, D tiles deep, waits for them with its own counter and
//     multiplies 16x16 blocks - no barrier until the end of K;
//   * the eight partial sums meet in LDS once (fixed order), then scale, bias, activation and gate;
//   * a row operation needs the whole row: the values go to an fp32 array in the workspace, and the
//     last M workgroups of the launch (one row each) wait for all others' arrival marks and run the
//     row op - or, where a launch may not wait (graph capture, FGE_FLAG_TWO_PASS), a second kernel
//     does.  Workgroups start in index order on each XCD, so with the device to itself a launch's waiting
//     workgroups have nobody behind them and need not be resident together with the rest of the grid.  A launch that
//     fills an XCD meanwhile may hold some back: the wait is bounded, and ends in NaN rows and the fault word.
#pragma once
#include "fge_device.h"

namespace fge {

constexpr int SKINNY_ROWS = 64;                       // rows the kernel takes
constexpr int SKINNY_WAVES = 8;

struct SkinnyArgs {
    const void *X, *W, *W2;                           // W2: second product of the gated form (else unused)
    const float *b, *b2, *gamma, *beta;
    void *out;
    float *aux;
    float *mid;                                       // row op: activated values, fp32, rows ld_mid apart
    unsigned *arrive;                                 // in-kernel row op: one arrival mark per workgroup
    int *fault;
    int M, N, K;
    int64_t ldx, ldw, ldo, ld_mid;
    float alpha, post, lo, hi, eps;
    int act, norm;
    int out_f32;                                      // results fp32 (else the 16-bit type of the operands)
    int in_kernel;                                    // the last workgroups run the row op
    unsigned gen, spin_limit;
    int withhold;                                     // tests only: workgroup 0 keeps its mark back
};

template <typename InT> struct SkinnyOut { typedef bf16_t type; };
template <> struct SkinnyOut<f16_t> { typedef f16_t type; };

// one 128-byte K tile of a 16 x 16 block: f[s] = chunk 4s + lane / 16 of row lane % 16 (both operands
// alike, so the sum over k is complete whatever k a slot holds)
// 16-bit operands: two sums, of the even and the odd 32 k, so that no chain of additions is longer than that of
// the tile kernels' K slices (64 x 8192 x 2048: relative error against float64 1.87e-7 as one sum, 1.44e-7 in K
// slices).  8-bit operands: one, whose error is that of the instruction (1.31e-5, with 64 terms per
// instruction as with 128).
template <typename InT> constexpr int SKINNY_SUMS = sizeof(InT) == 1 ? 1 : 2;
template <typename InT> __device__ __forceinline__ void skinny_mma(const u32x4 (&a)[2], const u32x4 (&b)[2], floatx4 (&sum)[SKINNY_SUMS<InT>]) {
    if constexpr (sizeof(InT) == 1) {
        floatx4 &c = sum[0];
        const i32x8 av = {(int)a[0].x, (int)a[0].y, (int)a[0].z, (int)a[0].w, (int)a[1].x, (int)a[1].y, (int)a[1].z, (int)a[1].w};
        const i32x8 bv = {(int)b[0].x, (int)b[0].y, (int)b[0].z, (int)b[0].w, (int)b[1].x, (int)b[1].y, (int)b[1].z, (int)b[1].w};
        c = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(av, bv, c, 0, 0, 0, 0, 0, 0);
    } else {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            floatx4 &c = sum[s];
            if constexpr (__is_same(InT, f16_t))
                c = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a[s]), __builtin_bit_cast(f16x8, b[s]), c, 0, 0, 0);
            else
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[s]), __builtin_bit_cast(bf16x8, b[s]), c, 0, 0, 0);
        }
    }
}

// The values of a row operation cross XCDs inside one launch: device-scope accesses on both sides.
__device__ __forceinline__ void skinny_put2(float *p, float v0, float v1) {
    __hip_atomic_store(reinterpret_cast<uint64_t *>(p), (uint64_t)as_u32(v0) | ((uint64_t)as_u32(v1) << 32), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 skinny_get2(const float *p) {
    const uint64_t bits = __hip_atomic_load(reinterpret_cast<const uint64_t *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return make_float2(as_f32((uint32_t)bits), as_f32((uint32_t)(bits >> 32)));
}

// The row operations read the row the workgroups left in mid.  The row stays in registers - NT threads
// hold up to 2*SKINNY_PAIRS*NT columns -, all its loads in flight together, and gamma / beta are
// fetched before the wait for the other workgroups (16 x 4096 x 4096 RMSNorm: 14.5 us when they were
// fetched behind it and the row went through LDS four loads at a time, 10.7 us so).
// (mid rows are an even number of floats; the element behind an odd row's last one is read, not used.)
constexpr int SKINNY_PAIRS = 8;
constexpr int SKINNY_ROW_N = 2 * SKINNY_PAIRS * 64 * SKINNY_WAVES;     // columns the product's own workgroups can finish
constexpr int SKINNY_WIDE_NT = 1024;                                   // threads of the row kernel for wider rows ...
constexpr int SKINNY_WIDE_N = 2 * SKINNY_PAIRS * SKINNY_WIDE_NT;       // ... and what they hold

struct SkinnyAffine { float2 g[SKINNY_PAIRS], b[SKINNY_PAIRS]; };       // of columns 2*(thread + NT*j), + 1

template <int NT> __device__ __forceinline__ void skinny_affine(const SkinnyArgs &a, SkinnyAffine &f) {
    const bool layer = a.norm == FGE_NORM_LAYERNORM, rms = a.norm == FGE_NORM_RMSNORM;
#pragma unroll
    for (int j = 0; j < SKINNY_PAIRS; ++j) {
        const int col = 2 * ((int)threadIdx.x + NT * j), c0 = min(col, a.N - 1), c1 = min(col + 1, a.N - 1);
        f.g[j] = make_float2(1.0f, 1.0f);
        f.b[j] = make_float2(0.0f, 0.0f);
        if ((layer || rms) && a.gamma != nullptr && col < a.N) f.g[j] = make_float2(a.gamma[c0], a.gamma[c1]);
        if (layer && a.beta != nullptr && col < a.N) f.b[j] = make_float2(a.beta[c0], a.beta[c1]);
    }
}

// Row operation on row `row`, one workgroup of NT threads.  groups: workgroups of the product (logsumexp
// merges one (maximum, sum) pair of each).  ok false: values are missing, the row becomes NaN.
template <typename NarrowT, int NT>
__device__ __forceinline__ void skinny_row(const SkinnyArgs &a, int row, int groups, const SkinnyAffine &aff, float (*red)[NT / 64], bool ok) {
    constexpr int NP = SKINNY_PAIRS;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float *src = a.mid + row * a.ld_mid;
    const float inv_n = 1.0f / (float)a.N;
    const float bad = ok ? 0.0f : __builtin_nanf("");
    int turn = 0;
    auto block_reduce = [&]<typename Op>(Op, float v) __attribute__((always_inline)) {
        v = allreduce64<Op>(v);
        if (lane == 0) red[turn][wave] = v;
        __syncthreads();
        float r = red[turn][0];
#pragma unroll
        for (int w = 1; w < NT / 64; ++w) r = Op::f(r, red[turn][w]);
        turn ^= 1;
        return r;
    };
    auto put = [&](int col, float v) __attribute__((always_inline)) {
        if (a.out_f32) Store<float>::put(reinterpret_cast<float *>(a.out) + row * a.ldo + col, v);
        else           Store<NarrowT>::put(reinterpret_cast<NarrowT *>(a.out) + row * a.ldo + col, v);
    };
    if (a.norm == FGE_NORM_LOGSUMEXP) {               // out holds the activated values already
        float m = OpMax::ident(), s = 0.0f;
        for (int p0 = tid; p0 < groups; p0 += NP * NT) {
            float2 e[NP];
#pragma unroll
            for (int j = 0; j < NP; ++j) e[j] = p0 + j * NT < groups ? skinny_get2(src + 2 * (p0 + j * NT)) : make_float2(OpMax::ident(), 0.0f);
            float mn = m;
#pragma unroll
            for (int j = 0; j < NP; ++j) mn = max_nc(mn, e[j].x);
            // (exp(-inf) = 0 drops a group of masked columns, but not the NaN its sum may be)
            const float r = exp_ref(mn);
            s *= fast_exp(m - r);
#pragma unroll
            for (int j = 0; j < NP; ++j) s += e[j].y * fast_exp(e[j].x - r);
            m = mn;
        }
        const float mt = m;
        m = block_reduce(OpMax{}, mt);
        s = block_reduce(OpSum{}, s * fast_exp(mt - exp_ref(m))) + bad;
        if (tid == 0) a.aux[row] = m + __logf(s);
        return;
    }
    const bool layer = a.norm == FGE_NORM_LAYERNORM;
    float2 v[NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        const int col = 2 * (tid + NT * j);
        v[j] = make_float2(0.0f, 0.0f);
        if (col < a.N) v[j] = skinny_get2(src + col);
    }
    if (a.norm == FGE_NORM_SOFTMAX) {
        float m = OpMax::ident();
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const int col = 2 * (tid + NT * j);
            if (col < a.N) m = max_nc(m, v[j].x);
            if (col + 1 < a.N) m = max_nc(m, v[j].y);
        }
        m = block_reduce(OpMax{}, m);
        const float c = -m * LOG2E;
        float s = 0.0f;
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const int col = 2 * (tid + NT * j);
            v[j] = make_float2(exp_rel(v[j].x, c), exp_rel(v[j].y, c));
            if (col < a.N) s += v[j].x;
            if (col + 1 < a.N) s += v[j].y;
        }
        const float inv = fast_rcp(block_reduce(OpSum{}, s) + bad);
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const int col = 2 * (tid + NT * j);
            if (col < a.N) put(col, v[j].x * inv);
            if (col + 1 < a.N) put(col + 1, v[j].y * inv);
        }
        return;
    }
    float shift = 0.0f, q2 = 0.0f;
    if (layer) {
        float sm = 0.0f;
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const int col = 2 * (tid + NT * j);
            if (col < a.N) sm += v[j].x;
            if (col + 1 < a.N) sm += v[j].y;
        }
        shift = block_reduce(OpSum{}, sm) * inv_n;
    }
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        const int col = 2 * (tid + NT * j);
        v[j] = make_float2(v[j].x - shift, v[j].y - shift);
        if (col < a.N) q2 += v[j].x * v[j].x;
        if (col + 1 < a.N) q2 += v[j].y * v[j].y;
    }
    const float rstd = rsqrtf(block_reduce(OpSum{}, q2) * inv_n + a.eps) + bad;
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        const int col = 2 * (tid + NT * j);
        if (col < a.N) put(col, v[j].x * rstd * aff.g[j].x + aff.b[j].x);
        if (col + 1 < a.N) put(col + 1, v[j].y * rstd * aff.g[j].y + aff.b[j].y);
    }
}

// MB: blocks of 16 rows (M <= 16*MB).  CB: blocks of 16 columns a workgroup multiplies - gated: one of
// each product.  D: K tiles in a wave's ring.
template <typename InT, int MB, int CB, bool GATED, int D>
__global__ __launch_bounds__(64 * SKINNY_WAVES) void skinny_kernel(const SkinnyArgs a) {
    static_assert(!GATED || CB == 2, "one column block of each product");
    typedef typename SkinnyOut<InT>::type NarrowT;
    constexpr int NT = 64 * SKINNY_WAVES;
    constexpr int STAGE = (MB + CB) * 2048;           // 16 rows x 128 bytes per block: X blocks, then W blocks
    constexpr int NS = 2 * (MB + CB);                 // copies per K tile
    constexpr int COLS = GATED ? 16 : 16 * CB;        // columns of the result per workgroup
    __shared__ __attribute__((aligned(16))) unsigned char smem[SKINNY_WAVES * D * STAGE];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n0 = blockIdx.x * COLS;
    const int row_bytes = a.K * (int)sizeof(InT);     // K tiles of 128 bytes; the last may be partial
    const int KT = (row_bytes + 127) >> 7;
    const int mine = (KT - wave + SKINNY_WAVES - 1) / SKINNY_WAVES;      // tiles wave, wave + 8, ... (KT >= 8: at least one)

    // ---------------- copies: copy i of a block fills rows 8i .. 8i+7 (lane l: row l / 8, physical chunk l % 8,
    // which holds global chunk (l % 8) ^ ((row / 2) % 8)); copy 1 uses the instruction offset 1024 for both
    // addresses, so its lane offset is lowered by as much
    constexpr int PRE = 1024;
    const int ld_r = lane >> 3, ld_c = lane & 7;
    const unsigned char *Xt = reinterpret_cast<const unsigned char *>(a.X) - PRE;
    const unsigned char *Wt = reinterpret_cast<const unsigned char *>(reinterpret_cast<const InT *>(a.W) + (int64_t)n0 * a.ldw) - PRE;
    const unsigned char *W2t = GATED ? reinterpret_cast<const unsigned char *>(reinterpret_cast<const InT *>(a.W2) + (int64_t)n0 * a.ldw) - PRE : Wt;
    uint32_t oX[MB][2], oW[CB][2];
    int chunk[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int r16 = i * 8 + ld_r;
        chunk[i] = ld_c ^ ((r16 >> 1) & 7);
        const uint32_t at = (uint32_t)(chunk[i] * 16 + PRE - i * 1024);
#pragma unroll
        for (int m = 0; m < MB; ++m) oX[m][i] = (uint32_t)((int64_t)min(m * 16 + r16, a.M - 1) * a.ldx) * (uint32_t)sizeof(InT) + at;
#pragma unroll
        for (int c = 0; c < CB; ++c)
            oW[c][i] = (uint32_t)((int64_t)(min(n0 + (GATED ? 0 : c * 16) + r16, a.N - 1) - n0) * a.ldw) * (uint32_t)sizeof(InT) + at;
    }
    unsigned char *ring = smem + wave * (D * STAGE);
    const uint32_t lds_ring = lds_address(smem) + (uint32_t)(wave * (D * STAGE));
    const bool ragged = (row_bytes & 127) != 0;
    // Where in its tiles a wave starts differs from workgroup to workgroup (the XCDs take them round robin).
    // Rows a power of two apart put the same K tile of every row of X and W on the same few L2 and
    // memory channels, and workgroups that walk K in step all ask those (32 x 8192 x 8192: 32.9 us in
    // step, 26.1 us so; 16 x 4096 x 4096 8.4 -> 8.1 us; no difference at other strides).
    int turn = (int)((blockIdx.x >> 3) + (blockIdx.x & 7)) % max(mine, 1);      // which of its tiles comes next
    auto copy_tile = [&](int t) __attribute__((always_inline)) {          // the t-th tile this wave takes
        const int kt = wave + turn * SKINNY_WAVES, buf = t % D;
        turn = turn + 1 == mine ? 0 : turn + 1;
        const int64_t k0 = (int64_t)kt * 128;
        uint64_t mask[2] = {~0ull, ~0ull};
        if (ragged && kt == KT - 1) {                 // lanes past K copy nothing, their chunks are zero
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const bool in = (int)k0 + chunk[i] * 16 < row_bytes;
                mask[i] = __ballot(in);
                if (!in) {
#pragma unroll
                    for (int q = 0; q < MB + CB; ++q)
                        *reinterpret_cast<u32x4 *>(ring + buf * STAGE + q * 2048 + i * 1024 + lane * 16) = u32x4{0u, 0u, 0u, 0u};
                }
            }
        }
#pragma unroll
        for (int c = 0; c < CB; ++c)
#pragma unroll
            for (int i = 0; i < 2; ++i)
                lds_dma16_masked((GATED && c == 1 ? W2t : Wt) + k0, oW[c][i], lds_ring + buf * STAGE + (MB + c) * 2048, i, i == 0, mask[i]);
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int i = 0; i < 2; ++i)
                lds_dma16_masked(Xt + k0, oX[m][i], lds_ring + buf * STAGE + m * 2048, i, i == 0, mask[i]);
    };

    floatx4 acc[MB][CB][SKINNY_SUMS<InT>];
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int c = 0; c < CB; ++c)
#pragma unroll
            for (int s = 0; s < SKINNY_SUMS<InT>; ++s) acc[m][c][s] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    const int f_row = lane & 15, f_q = lane >> 4;
    int fo[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) fo[s] = f_row * 128 + (((4 * s + f_q) ^ ((f_row >> 1) & 7)) << 4);

#pragma unroll
    for (int t = 0; t < D; ++t)
        if (t < mine) copy_tile(t);
    for (int t = 0; t < mine; ++t) {
        // copies complete in issue order: tile t has landed when only those of later tiles are out
        const int later = min(mine - 1 - t, D - 1);
        if (D > 3 && later == 3)      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(3 * NS) : "memory");
        else if (D > 2 && later == 2) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(2 * NS) : "memory");
        else if (D > 1 && later == 1) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(NS) : "memory");
        else                          asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        const unsigned char *st = ring + (t % D) * STAGE;
        u32x4 fx[MB][2], fw[CB][2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
#pragma unroll
            for (int c = 0; c < CB; ++c) fw[c][s] = *reinterpret_cast<const u32x4 *>(st + (MB + c) * 2048 + fo[s]);
#pragma unroll
            for (int m = 0; m < MB; ++m) fx[m][s] = *reinterpret_cast<const u32x4 *>(st + m * 2048 + fo[s]);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");    // the fragments are in registers: the buffer is free
        __builtin_amdgcn_sched_barrier(0);
        if (t + D < mine) copy_tile(t + D);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int c = 0; c < CB; ++c) skinny_mma<InT>(fx[m], fw[c], acc[m][c]);
    }

    // ---------------- the eight partial sums, added in wave order.  Block layout: element (row, col) in
    // lane (row / 4) * 16 + col, register row % 4.
    static_assert(MB * CB * 1024 <= D * STAGE, "partial sums fit the ring");
    {
        float *mine_f = reinterpret_cast<float *>(ring);
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int c = 0; c < CB; ++c) {
                floatx4 v = acc[m][c][0];
#pragma unroll
                for (int s = 1; s < SKINNY_SUMS<InT>; ++s)
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] += acc[m][c][s][e];
                *reinterpret_cast<floatx4 *>(mine_f + (m * CB + c) * 256 + lane * 4) = v;
            }
    }
    __syncthreads();
    const float *sums = reinterpret_cast<const float *>(smem);
    const float scale = a.post * a.alpha;
    constexpr int ITEMS = MB * 16 * COLS / 2;         // two neighbouring columns each
#pragma unroll
    for (int it = 0; it < (ITEMS + NT - 1) / NT; ++it) {
        const int e = tid + it * NT;
        const int row = e / (COLS / 2), cc = (e % (COLS / 2)) * 2, col = n0 + cc;
        if (e >= ITEMS || row >= a.M) continue;       // (uniform over the lanes that share a row)
        float v[2], u[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int c16 = (cc + j) & 15, r16 = row & 15;
            const int at = ((r16 >> 2) * 16 + c16) * 4 + (r16 & 3), blk = (row >> 4) * CB;
            float s = 0.0f, s2 = 0.0f;
#pragma unroll
            for (int w = 0; w < SKINNY_WAVES; ++w) {
                const float *f = sums + w * (D * STAGE / 4);
                s += f[(blk + (GATED ? 0 : (cc + j) >> 4)) * 256 + at];
                if constexpr (GATED) s2 += f[(blk + 1) * 256 + at];
            }
            const int cj = min(col + j, a.N - 1);
            v[j] = scale * s + (a.b != nullptr ? a.post * a.b[cj] : 0.0f);
            u[j] = GATED ? scale * s2 + (a.b2 != nullptr ? a.post * a.b2[cj] : 0.0f) : 1.0f;
        }
        dispatch_act(a.act, [&]<int ACT>() __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < 2; ++j) v[j] = activate<ACT>(v[j], a.lo, a.hi) * u[j];
        });
        if (a.norm == FGE_NORM_LOGSUMEXP) {           // maximum and sum of exponentials over this workgroup's columns
            const float v1 = col + 1 < a.N ? v[1] : OpMax::ident();
            const float m = allreduce_lanes<OpMax, COLS / 2>(col < a.N ? max_nc(v[0], v1) : OpMax::ident());
            const float r = exp_ref(m);               // (the columns may all be masked, by any value)
            const float s = allreduce_lanes<OpSum, COLS / 2>(col < a.N ? exp_diff(v[0], r) + (col + 1 < a.N ? exp_diff(v[1], r) : 0.0f) : 0.0f);
            if (cc == 0) skinny_put2(a.mid + row * a.ld_mid + 2 * blockIdx.x, m, s);
        } else if (a.norm != FGE_NORM_NONE && col < a.N) {
            skinny_put2(a.mid + row * a.ld_mid + col, v[0], v[1]);
        }
        if (a.norm == FGE_NORM_NONE || a.norm == FGE_NORM_LOGSUMEXP) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                if (col + j >= a.N) continue;
                if (a.out_f32) Store<float>::put(reinterpret_cast<float *>(a.out) + row * a.ldo + col + j, v[j]);
                else           Store<NarrowT>::put(reinterpret_cast<NarrowT *>(a.out) + row * a.ldo + col + j, v[j]);
            }
        }
    }
    if (!a.in_kernel) return;

    // ---------------- row operation by the last workgroups
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's values have reached the device-coherent level
    __syncthreads();                                  // ... every wave's; the partial sums are consumed
    const int G = gridDim.x, F = min(a.M, G);
    if (tid == 0 && !(a.withhold && blockIdx.x == 0))
        __hip_atomic_store(a.arrive + blockIdx.x, a.gen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int f = (int)blockIdx.x - (G - F);
    if (f < 0) return;
    SkinnyAffine aff;
    skinny_affine<NT>(a, aff);
    bool ok = true;
    for (int t = tid; t < G; t += NT) {
        unsigned spins = 0;
        while (__hip_atomic_load(a.arrive + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != a.gen) {
            __builtin_amdgcn_s_sleep(4);
            if (++spins > a.spin_limit) { ok = false; break; }
        }
    }
    float (*red)[SKINNY_WAVES] = reinterpret_cast<float (*)[SKINNY_WAVES]>(smem);
    if (lane == 0) red[0][wave] = __all(ok) ? 1.0f : 0.0f;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < SKINNY_WAVES; ++w) ok = ok && red[0][w] != 0.0f;
    if (!ok && tid == 0) *a.fault = 1;
    for (int row = f; row < a.M; row += F) {
        __syncthreads();
        skinny_row<NarrowT, NT>(a, row, G, aff, red, ok);
    }
}

// The row operation as a kernel of its own: one workgroup per row.
template <typename NarrowT, int NT>
__global__ __launch_bounds__(NT) void skinny_rows_kernel(const SkinnyArgs a, int groups) {
    __shared__ float red[2][NT / 64];
    SkinnyAffine aff;
    skinny_affine<NT>(a, aff);
    skinny_row<NarrowT, NT>(a, blockIdx.x, groups, aff, red, true);
}

}  // namespace fge
