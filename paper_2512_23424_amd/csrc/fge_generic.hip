// Element-granular kernels for shapes the vectorised kernels do not take: extents or strides
// that are not multiples of 16 bytes, and row operations over rows wider than a wave's
// registers hold.  They make every valid shape computable (fp32 products and sums, scalar loads and
// stores, rows re-read from memory per pass).
//
//   generic_gemm_kernel : dst = act(post*(alpha*X.W^T + b))   32x32 tile, LDS staged, fp32 matrix instruction
//   generic_act_kernel  : dst = act(src) [* second operand]   elementwise
//   any_row_kernel      : out = rowop(src)                    rows of up to 8192 columns but the shortest, in registers
//   generic_row_kernel  : out = rowop(src)                    other rows: one wave per row, passes over src
//   splitk_sum_kernel   : dst = act(post*(alpha*sum_s P_s + b))  the slices of a K-split product, summed in slice order
//   pad_rows_kernel     : dense copy of a matrix with K padded by zeros to whole 16-byte chunks
//                         (and zero rows appended): what makes an operand with odd extents or
//                         strides fit the vectorised kernels, at one extra read and write of it
#include "fge_launch.h"

namespace fge {

namespace {

template <typename T> __device__ __forceinline__ const T *row_ptr(const void *base, int64_t rowg, int M,
                                                                 int64_t ld, int64_t bs) {
    return reinterpret_cast<const T *>(base) + (rowg / M) * bs + (rowg % M) * ld;
}

// A 32x32 tile of outputs per workgroup.  Small problems of odd extents are its work, so what bounds it is a chain of
// memory latencies along K: KT = 128 k are fetched at a time, one K tile ahead in registers, and the four waves share out each
// K tile (32 k each, fp32 matrix instruction) and add their sums in LDS.  (32 k at a time, nothing
// ahead, an FMA per value read from LDS: 365 x 429 x 32 SiLU LayerNorm 35.8 us, now 12.1;
// 17 x 500 x 33 34.9 and 8.7, 40 x 64 x 47 LayerNorm 9.9 and 8.8.)  A K of up to 32 or 64 is one tile of that many k: staging 128
// cost calls of a few microseconds up to a third (f16 1 x 31 x 145, with 128, now, with that former kernel: 4.3, 2.7, 3.6).
template <typename InT, typename DstT, int KT>
__global__ __launch_bounds__(256) void generic_gemm_kernel(const GenArgs a) {
    constexpr int T = 32, LD = KT + 4, STEP = 256 / KT, RPT = T / STEP;   // LD: rows 16-byte aligned, four banks apart
    constexpr int PANELS = 2 * T * LD, SUMS = 4 * T * T;
    __shared__ __attribute__((aligned(16))) float xs[PANELS > SUMS ? PANELS : SUMS];
    float *ws = xs + T * LD;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, h = lane >> 5;
    const int n0 = blockIdx.x * T, m0 = blockIdx.y * T, z = blockIdx.z;
    const InT *X = reinterpret_cast<const InT *>(a.X) + (int64_t)z * a.bsx;
    const InT *W = reinterpret_cast<const InT *>(a.W);
    const int lk = tid & (KT - 1), lr = tid / KT;                    // this thread's k and first row of a K tile
    InT xr[RPT], wr[RPT];                                            // as they lie in memory: a conversion behind each load would wait for it
    auto fetch = [&](int k0) __attribute__((always_inline)) {
        const int k = k0 + lk;
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const int r = lr + STEP * i;
            xr[i] = (m0 + r < a.M && k < a.K) ? X[(int64_t)(m0 + r) * a.ldx + k] : InT{};
            wr[i] = (n0 + r < a.N && k < a.K) ? W[(int64_t)(n0 + r) * a.ldw + k] : InT{};
        }
    };
    floatx16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
    fetch(0);
    for (int k0 = 0; k0 < a.K; k0 += KT) {
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            xs[(lr + STEP * i) * LD + lk] = Store<InT>::get(&xr[i]);
            ws[(lr + STEP * i) * LD + lk] = Store<InT>::get(&wr[i]);
        }
        __syncthreads();
        if (k0 + KT < a.K) fetch(k0 + KT);
#pragma unroll
        for (int u = 0; u < KT / 32; ++u) {                          // lanes 0-31: k 8u .. 8u+3 of the wave's, lanes 32-63: the next four
            const int at = l32 * LD + wave * (KT / 4) + u * 8 + h * 4;
            Mma<float>::run(*reinterpret_cast<const u32x4 *>(xs + at), *reinterpret_cast<const u32x4 *>(ws + at), acc);
        }
        __syncthreads();
    }
    // the waves' sums: [wave][row][column], 32 floats a row, in the panels' place
#pragma unroll
    for (int r = 0; r < 16; ++r) xs[wave * T * T + ((r >> 2) * 8 + h * 4 + (r & 3)) * T + l32] = acc[r];
    __syncthreads();
    const int tx = tid & 31, ty = tid >> 5;
    const int col = n0 + tx;
    if (col >= a.N) return;
    const float scale = a.post * a.alpha;
    const float bias = a.b != nullptr ? a.post * a.b[col] : 0.0f;
    DstT *dst = reinterpret_cast<DstT *>(a.dst) + (int64_t)z * a.bsd;
    dispatch_act(a.act, [&]<int ACT>() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = ty + 8 * i, row = m0 + r;
            const float *p = xs + r * T + tx;
            const float sum = (p[0] + p[T * T]) + (p[2 * T * T] + p[3 * T * T]);
            if (row < a.M)
                Store<DstT>::put(dst + (int64_t)row * a.ldd + col, activate<ACT>(scale * sum + bias, a.lo, a.hi));
        }
    });
}

template <typename T>
__global__ __launch_bounds__(256) void generic_act_kernel(const GenArgs a) {
    const int64_t total = (int64_t)a.batch * a.M * a.N;
    dispatch_act(a.act, [&]<int ACT>() __attribute__((always_inline)) {
        for (int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (int64_t)gridDim.x * 256) {
            const int64_t rowg = idx / a.N;
            const int c = (int)(idx - rowg * a.N);
            const int64_t off = (rowg / a.M) * a.bsd + (rowg % a.M) * a.ldd + c;
            float v = activate<ACT>(Store<T>::get(reinterpret_cast<const T *>(a.X) + off), a.lo, a.hi);
            if (a.W != nullptr) v *= Store<T>::get(reinterpret_cast<const T *>(a.W) + off);   // gate
            Store<T>::put(reinterpret_cast<T *>(a.dst) + off, v);
        }
    });
}

// The same on rows that registers hold (see launch_generic_row): WAVES waves per row, NCH chunks of CW values per lane, loaded and
// stored 16 bytes at a time at any alignment and read once.  (The kernel below reads a value at a time, three times over; us, with it
// -> so, floor at a large copy's 5.8 TB/s: bf16 65536 x 4095 RMSNorm 520.6 -> 306.2 / 185, 65536 x 2047 softmax 356.7 -> 171.8 / 93, fp32 65536 x 2047
// LayerNorm 436.9 -> 201.6 / 185, 9000 x 8191 RMSNorm 275.1 -> 110.7 / 102, f16 4000 x 8191 logsumexp 120.8 -> 34.5 / 23.  What is left in 16
// bits is the rows' halves of sectors, written by two workgroups.)
template <typename SrcT, typename OutT, int WAVES, int NCH>
__global__ __launch_bounds__(256) void any_row_kernel(const GenArgs a) {
    constexpr int CW = Store<OutT>::CW, SL = CW / Store<SrcT>::CW;      // values per chunk; loads per chunk
    static_assert(SL >= 1, "source no narrower than the result");
    constexpr int TEAM = 64 * WAVES;
    __shared__ float red[2][4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int member = WAVES == 1 ? lane : (int)threadIdx.x;
    const int64_t rowg = WAVES == 1 ? (int64_t)blockIdx.x * 4 + wave : (int64_t)blockIdx.x;
    if (rowg >= (int64_t)a.batch * a.M) return;                       // wave-uniform (WAVES = 4: never)
    const SrcT *src = row_ptr<SrcT>(a.X, rowg, a.M, a.ldx, a.bsx);
    OutT *out = const_cast<OutT *>(row_ptr<OutT>(a.dst, rowg, a.M, a.ldd, a.bsd));
    const bool in_place = reinterpret_cast<const void *>(src) == reinterpret_cast<const void *>(out);
    if (a.norm == FGE_NORM_NONE && in_place) return;                  // nothing to do: no value is written back
    const float inv_n = 1.0f / (float)a.N;
    int turn = 0;
    auto reduce = [&]<typename Op>(Op, float v) __attribute__((always_inline)) {
        v = allreduce64<Op>(v);
        if constexpr (WAVES > 1) {
            if (lane == 0) red[turn][wave] = v;
            __syncthreads();
            v = Op::f(Op::f(red[turn][0], red[turn][1]), Op::f(red[turn][2], red[turn][3]));
            turn ^= 1;
        }
        return v;
    };
    float v[NCH][CW];
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        const int j0 = (c * TEAM + member) * CW;
        if (j0 + CW <= a.N) {
#pragma unroll
            for (int l = 0; l < SL; ++l) {
                typedef typename Store<SrcT>::any16 chunk_t;
                const u32x4 u = *reinterpret_cast<const chunk_t *>(src + j0 + l * Store<SrcT>::CW);
                Store<SrcT>::unpack(make_uint4(u.x, u.y, u.z, u.w), v[c] + l * Store<SrcT>::CW);
            }
        } else {
            SrcT tail[CW];                                           // (converted behind all the loads: each conversion waits for its own)
#pragma unroll
            for (int e = 0; e < CW; ++e) tail[e] = j0 + e < a.N ? src[j0 + e] : SrcT{};
#pragma unroll
            for (int e = 0; e < CW; ++e) v[c][e] = Store<SrcT>::get(tail + e);
        }
    }
    auto each = [&](auto &&f) __attribute__((always_inline)) {           // f(value, column) for the row's own values
#pragma unroll
        for (int c = 0; c < NCH; ++c)
#pragma unroll
            for (int e = 0; e < CW; ++e) {
                const int j = (c * TEAM + member) * CW + e;
                if (j < a.N) f(v[c][e], j);
            }
    };
    // f(value, gamma, beta): the vectors start on 16-byte boundaries, and so do a chunk's parts of them
    auto part = [&](const float *p, int j, float none) __attribute__((always_inline)) {
        floatx4 r = {none, none, none, none};
        if (p == nullptr) return r;
        if (j + 4 <= a.N) return *reinterpret_cast<const floatx4 *>(p + j);
#pragma unroll
        for (int e = 0; e < 3; ++e)
            if (j + e < a.N) r[e] = p[j + e];
        return r;
    };
    auto affine = [&](auto &&f) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < NCH; ++c)
#pragma unroll
            for (int e = 0; e < CW; e += 4) {
                const int j = (c * TEAM + member) * CW + e;
                const floatx4 g = part(a.gamma, j, 1.0f), b = part(a.norm == FGE_NORM_LAYERNORM ? a.beta : nullptr, j, 0.0f);
#pragma unroll
                for (int i = 0; i < 4; ++i) f(v[c][e + i], g[i], b[i]);
            }
    };
    if (a.norm == FGE_NORM_SOFTMAX || a.norm == FGE_NORM_LOGSUMEXP) {
        float m = OpMax::ident();
        each([&](float &x, int) __attribute__((always_inline)) { m = max_nc(m, x); });
        m = reduce(OpMax{}, m);
        float s = 0.0f;
        if (a.norm == FGE_NORM_SOFTMAX) {
            each([&](float &x, int) __attribute__((always_inline)) { x = fast_exp(x - m); s += x; });
            const float inv = 1.0f / reduce(OpSum{}, s);
            each([&](float &x, int) __attribute__((always_inline)) { x *= inv; });
        } else {
            each([&](float &x, int) __attribute__((always_inline)) { s += fast_exp(x - m); });
            s = reduce(OpSum{}, s);
            if (member == 0) a.aux[rowg] = m + __logf(s);
            if (in_place) return;
        }
    } else if (a.norm == FGE_NORM_LAYERNORM) {
        float s = 0.0f, d2 = 0.0f;
        each([&](float &x, int) __attribute__((always_inline)) { s += x; });
        const float mean = reduce(OpSum{}, s) * inv_n;
        each([&](float &x, int) __attribute__((always_inline)) { x -= mean; d2 += x * x; });
        const float rstd = rsqrtf(reduce(OpSum{}, d2) * inv_n + a.eps);
        affine([&](float &x, float g, float b) __attribute__((always_inline)) { x = x * rstd * g + b; });
    } else if (a.norm == FGE_NORM_RMSNORM) {
        float s = 0.0f;
        each([&](float &x, int) __attribute__((always_inline)) { s += x * x; });
        const float rr = rsqrtf(reduce(OpSum{}, s) * inv_n + a.eps);
        affine([&](float &x, float g, float) __attribute__((always_inline)) { x *= rr * g; });
    }
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        const int j0 = (c * TEAM + member) * CW;
        if (j0 + CW <= a.N) {
            const uint4 u = Store<OutT>::pack(v[c]);
            const u32x4 w = {u.x, u.y, u.z, u.w};
            *reinterpret_cast<typename Store<OutT>::any16 *>(out + j0) = w;
        } else {
#pragma unroll
            for (int e = 0; e < CW; ++e)
                if (j0 + e < a.N) Store<OutT>::put(out + j0 + e, v[c][e]);
        }
    }
}

// src: rows x N of SrcT (row stride lds, batch stride bss); out: rows x N of OutT (ldd, bsd).
template <typename SrcT, typename OutT>
__global__ __launch_bounds__(256) void generic_row_kernel(const GenArgs a) {
    const int lane = threadIdx.x & 63;
    const int64_t rowg = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (rowg >= (int64_t)a.batch * a.M) return;                       // wave-uniform
    const SrcT *src = row_ptr<SrcT>(a.X, rowg, a.M, a.ldx, a.bsx);
    OutT *out = const_cast<OutT *>(row_ptr<OutT>(a.dst, rowg, a.M, a.ldd, a.bsd));
    const float inv_n = 1.0f / (float)a.N;
    if (a.norm == FGE_NORM_SOFTMAX || a.norm == FGE_NORM_LOGSUMEXP) {
        float m = OpMax::ident();
        for (int j = lane; j < a.N; j += 64) m = max_nc(m, Store<SrcT>::get(src + j));
        m = allreduce64<OpMax>(m);
        float s = 0.0f;
        for (int j = lane; j < a.N; j += 64) s += fast_exp(Store<SrcT>::get(src + j) - m);
        s = allreduce64<OpSum>(s);
        if (a.norm == FGE_NORM_SOFTMAX) {
            const float inv = 1.0f / s;
            for (int j = lane; j < a.N; j += 64) Store<OutT>::put(out + j, fast_exp(Store<SrcT>::get(src + j) - m) * inv);
        } else {
            if (lane == 0) a.aux[rowg] = m + __logf(s);
            if (reinterpret_cast<const void *>(src) != reinterpret_cast<const void *>(out))
                for (int j = lane; j < a.N; j += 64) Store<OutT>::put(out + j, Store<SrcT>::get(src + j));
        }
    } else if (a.norm == FGE_NORM_LAYERNORM) {
        float s = 0.0f;
        for (int j = lane; j < a.N; j += 64) s += Store<SrcT>::get(src + j);
        const float mean = allreduce64<OpSum>(s) * inv_n;
        float d2 = 0.0f;
        for (int j = lane; j < a.N; j += 64) {
            const float d = Store<SrcT>::get(src + j) - mean;
            d2 += d * d;
        }
        const float rstd = rsqrtf(allreduce64<OpSum>(d2) * inv_n + a.eps);
        for (int j = lane; j < a.N; j += 64) {
            const float g = a.gamma != nullptr ? a.gamma[j] : 1.0f, b = a.beta != nullptr ? a.beta[j] : 0.0f;
            Store<OutT>::put(out + j, (Store<SrcT>::get(src + j) - mean) * rstd * g + b);
        }
    } else if (a.norm == FGE_NORM_RMSNORM) {
        float s = 0.0f;
        for (int j = lane; j < a.N; j += 64) {
            const float v = Store<SrcT>::get(src + j);
            s += v * v;
        }
        const float rr = rsqrtf(allreduce64<OpSum>(s) * inv_n + a.eps);
        for (int j = lane; j < a.N; j += 64) {
            const float g = a.gamma != nullptr ? a.gamma[j] : 1.0f;
            Store<OutT>::put(out + j, Store<SrcT>::get(src + j) * rr * g);
        }
    } else {
        if (reinterpret_cast<const void *>(src) != reinterpret_cast<const void *>(out))
            for (int j = lane; j < a.N; j += 64) Store<OutT>::put(out + j, Store<SrcT>::get(src + j));
    }
}

// The same row operation for fp32 source rows that start on 16-byte boundaries (the rows of padded
// width the repacked path produces; ldx and bsx multiples of 4) and a result of any width and
// stride: one workgroup of four waves per row.  The statistics passes read 16 bytes per lane, four
// loads in flight per thread; the last pass reads and writes one element per lane, so that a
// wave's stores are one contiguous run whatever the alignment of the result's rows.  CACHE: the
// row (at most 64 KB) is parked in LDS by the first pass and read from there afterwards; longer
// rows are read from memory by every pass, and softmax / logsumexp take their two statistics in
// one pass.
// (The wave-per-row kernel above walks a row with one load in flight per lane: 2048 rows of 50257
// columns took it 1.0 ms.)
template <typename OutT, bool CACHE>
__global__ __launch_bounds__(256) void aligned_src_row_kernel(const GenArgs a) {
    __shared__ float red[2][4];
    extern __shared__ __attribute__((aligned(16))) float rowbuf[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t rowg = blockIdx.x;
    const float *src = row_ptr<float>(a.X, rowg, a.M, a.ldx, a.bsx);
    OutT *out = const_cast<OutT *>(row_ptr<OutT>(a.dst, rowg, a.M, a.ldd, a.bsd));
    const int n4 = a.N >> 2;                                     // whole groups of four columns
    const float inv_n = 1.0f / (float)a.N;
    int turn = 0;
    auto block_reduce = [&]<typename Op>(Op, float v) __attribute__((always_inline)) {
        v = allreduce64<Op>(v);
        if (lane == 0) red[turn][wave] = v;
        __syncthreads();
        const float r = Op::f(Op::f(red[turn][0], red[turn][1]), Op::f(red[turn][2], red[turn][3]));
        turn ^= 1;
        return r;
    };
    // first pass over the row: f(v) for every valid element, 16 bytes per lane (+ the ragged tail)
    auto sweep_first = [&](auto &&f) __attribute__((always_inline)) {
#pragma unroll 4
        for (int q = tid; q < n4; q += 256) {
            const floatx4 v = *reinterpret_cast<const floatx4 *>(src + 4 * q);
            if constexpr (CACHE) *reinterpret_cast<floatx4 *>(rowbuf + 4 * q) = v;
            f(v[0]); f(v[1]); f(v[2]); f(v[3]);
        }
        const int j = 4 * n4 + tid;
        if (j < a.N) {
            const float v = src[j];
            if constexpr (CACHE) rowbuf[j] = v;
            f(v);
        }
        if constexpr (CACHE) __syncthreads();
    };
    auto sweep = [&](auto &&f) __attribute__((always_inline)) {
        const float *r = CACHE ? rowbuf : src;
#pragma unroll 4
        for (int q = tid; q < n4; q += 256) {
            const floatx4 v = *reinterpret_cast<const floatx4 *>(r + 4 * q);
            f(v[0]); f(v[1]); f(v[2]); f(v[3]);
        }
        const int j = 4 * n4 + tid;
        if (j < a.N) f(r[j]);
    };
    // last pass: out[j] = g(j, v[j]), one element per lane and step
    auto emit = [&](auto &&g) __attribute__((always_inline)) {
        const float *r = CACHE ? rowbuf : src;
#pragma unroll 4
        for (int j = tid; j < a.N; j += 256) Store<OutT>::put(out + j, g(j, r[j]));
    };
    if (a.norm == FGE_NORM_SOFTMAX || a.norm == FGE_NORM_LOGSUMEXP) {
        float m = OpMax::ident(), s = 0.0f, c;
        if constexpr (CACHE) {
            sweep_first([&](float v) __attribute__((always_inline)) { m = max_nc(m, v); });
            m = block_reduce(OpMax{}, m);
            c = -m * LOG2E;
            sweep([&](float v) __attribute__((always_inline)) { s += exp_rel(v, c); });
            s = block_reduce(OpSum{}, s);
        } else {
            // a row that is read from memory every time: maximum and sum in one pass - every thread
            // keeps a running maximum and rescales its sum so far whenever the maximum rises (the values
            // so far may all be masked, by any value: see exp_diff; a thread without elements ends with
            // 0 * exp2(-inf) = 0)
#pragma unroll 4
            for (int q = tid; q < n4; q += 256) {
                const floatx4 v = *reinterpret_cast<const floatx4 *>(src + 4 * q);
                const float mn = max_nc(max_nc(max_nc(v[0], v[1]), max_nc(v[2], v[3])), m);
                const float r = exp_ref(mn);
                s = s * exp_diff(m, r) + ((exp_diff(v[0], r) + exp_diff(v[1], r)) + (exp_diff(v[2], r) + exp_diff(v[3], r)));
                m = mn;
            }
            if (const int j = 4 * n4 + tid; j < a.N) {
                const float v = src[j], mn = max_nc(v, m), r = exp_ref(mn);
                s = s * exp_diff(m, r) + exp_diff(v, r);
                m = mn;
            }
            const float mt = m;
            m = block_reduce(OpMax{}, mt);
            c = -m * LOG2E;
            s = block_reduce(OpSum{}, s * exp_diff(mt, exp_ref(m)));
        }
        if (a.norm == FGE_NORM_SOFTMAX) {
            const float inv = 1.0f / s;
            emit([&](int, float v) __attribute__((always_inline)) { return exp_rel(v, c) * inv; });
        } else {
            if (tid == 0) a.aux[rowg] = m + __logf(s);
            emit([&](int, float v) __attribute__((always_inline)) { return v; });
        }
    } else if (a.norm == FGE_NORM_LAYERNORM) {
        float s = 0.0f;
        sweep_first([&](float v) __attribute__((always_inline)) { s += v; });
        const float mean = block_reduce(OpSum{}, s) * inv_n;
        float d2 = 0.0f;
        sweep([&](float v) __attribute__((always_inline)) { d2 += (v - mean) * (v - mean); });
        const float rstd = rsqrtf(block_reduce(OpSum{}, d2) * inv_n + a.eps);
        emit([&](int j, float v) __attribute__((always_inline)) {
            return (v - mean) * rstd * (a.gamma != nullptr ? a.gamma[j] : 1.0f) + (a.beta != nullptr ? a.beta[j] : 0.0f);
        });
    } else if (a.norm == FGE_NORM_RMSNORM) {
        float s = 0.0f;
        sweep_first([&](float v) __attribute__((always_inline)) { s += v * v; });
        const float rr = rsqrtf(block_reduce(OpSum{}, s) * inv_n + a.eps);
        emit([&](int j, float v) __attribute__((always_inline)) { return v * rr * (a.gamma != nullptr ? a.gamma[j] : 1.0f); });
    } else {
        sweep_first([&](float) __attribute__((always_inline)) {});
        emit([&](int, float v) __attribute__((always_inline)) { return v; });
    }
}

// K-split product: X holds `K` dense fp32 slices of M x N partial sums, `bsx` elements apart; four
// neighbouring columns per thread (N is a multiple of 4).  The slices are added in slice order,
// so the result does not depend on how the launch was scheduled.
template <typename DstT>
__global__ __launch_bounds__(256) void splitk_sum_kernel(const GenArgs a) {
    const int n4 = a.N >> 2;
    const int64_t total = (int64_t)a.M * n4;
    const float *P = reinterpret_cast<const float *>(a.X);
    const float *P2 = reinterpret_cast<const float *>(a.W);     // gated form: the second product's slices
    const float scale = a.post * a.alpha;
    auto sum = [&](const float *q) __attribute__((always_inline)) {
        floatx4 acc = *reinterpret_cast<const floatx4 *>(q);
        for (int sl = 1; sl < a.K; ++sl) {
            const floatx4 v = *reinterpret_cast<const floatx4 *>(q + sl * a.bsx);
            acc[0] += v[0]; acc[1] += v[1]; acc[2] += v[2]; acc[3] += v[3];
        }
        return acc;
    };
    dispatch_act(a.act, [&]<int ACT>() __attribute__((always_inline)) {
        for (int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (int64_t)gridDim.x * 256) {
            const int64_t row = idx / n4;
            const int col = (int)(idx - row * n4) << 2;
            const floatx4 acc = sum(P + row * a.N + col);
            floatx4 gate = {1.0f, 1.0f, 1.0f, 1.0f};
            if (P2 != nullptr) {
                const floatx4 u = sum(P2 + row * a.N + col);
#pragma unroll
                for (int e = 0; e < 4; ++e) gate[e] = scale * u[e] + (a.b2 != nullptr ? a.post * a.b2[col + e] : 0.0f);
            }
            DstT *d = reinterpret_cast<DstT *>(a.dst) + row * a.ldd + col;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float bias = a.b != nullptr ? a.post * a.b[col + e] : 0.0f;
                Store<DstT>::put(d + e, activate<ACT>(scale * acc[e] + bias, a.lo, a.hi) * gate[e]);
            }
        }
    });
}

// dst: rows_dst x Kp dense (Kp a multiple of the 16-byte chunk); row r < batch * M is row r of the
// source (M rows per problem, strides ld / bs), zero filled from K on; rows beyond are zero.
// One thread per 16-byte chunk of dst: element-granular reads (the source rows need not be
// aligned), one 16-byte store.
template <typename T>
__global__ __launch_bounds__(256) void pad_rows_kernel(const PadArgs a) {
    constexpr int CW = 16 / (int)sizeof(T);
    const int cpr = a.Kp / CW;
    const int64_t total = a.rows_dst * cpr;
    for (int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (int64_t)gridDim.x * 256) {
        const int64_t r = idx / cpr;
        const int k0 = (int)(idx - r * cpr) * CW;
        T v[CW];
        const bool live = r < (int64_t)a.batch * a.M;
        const T *src = live ? row_ptr<T>(a.src, r, a.M, a.ld, a.bs) : nullptr;
#pragma unroll
        for (int e = 0; e < CW; ++e) {
            T z{};
            v[e] = (live && k0 + e < a.K) ? src[k0 + e] : z;
        }
        *reinterpret_cast<uint4 *>(reinterpret_cast<T *>(a.dst) + r * a.Kp + k0) = *reinterpret_cast<const uint4 *>(v);
    }
}

// dst[0 .. np) = src[0 .. n), zero beyond
__global__ __launch_bounds__(256) void pad_vec_kernel(const float *src, float *dst, int n, int np) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < np) dst[i] = i < n ? src[i] : 0.0f;
}

}  // namespace

hipError_t launch_pad_rows(int dtype, hipStream_t s, const PadArgs &a) {
    const int cw = dtype == FGE_F32 ? 4 : dtype == FGE_F8E4M3 ? 16 : 8;
    const int64_t total = a.rows_dst * (a.Kp / cw);
    int64_t blocks = (total + 255) / 256;
    if (blocks > 256 * 64) blocks = 256 * 64;                           // grid-stride beyond that
    const dim3 grid((unsigned)(blocks > 0 ? blocks : 1)), block(256);
    if (dtype == FGE_F32)          hipLaunchKernelGGL((pad_rows_kernel<float>), grid, block, 0, s, a);
    else if (dtype == FGE_F8E4M3)  hipLaunchKernelGGL((pad_rows_kernel<f8_t>), grid, block, 0, s, a);
    else                           hipLaunchKernelGGL((pad_rows_kernel<bf16_t>), grid, block, 0, s, a);   // any 16-bit type: bits are copied
    return hipGetLastError();
}

hipError_t launch_pad_vec(const float *src, float *dst, int n, int np, hipStream_t s) {
    hipLaunchKernelGGL(pad_vec_kernel, dim3((unsigned)((np + 255) / 256)), dim3(256), 0, s, src, dst, n, np);
    return hipGetLastError();
}

hipError_t launch_splitk_sum(int dst_dtype, hipStream_t s, const GenArgs &a) {
    const int64_t total = (int64_t)a.M * (a.N >> 2);
    int64_t blocks = (total + 255) / 256;
    if (blocks > 256 * 32) blocks = 256 * 32;                           // grid-stride beyond that
    const dim3 grid((unsigned)blocks), block(256);
    if (dst_dtype == FGE_BF16)     hipLaunchKernelGGL((splitk_sum_kernel<bf16_t>), grid, block, 0, s, a);
    else if (dst_dtype == FGE_F16) hipLaunchKernelGGL((splitk_sum_kernel<f16_t>), grid, block, 0, s, a);
    else                           hipLaunchKernelGGL((splitk_sum_kernel<float>), grid, block, 0, s, a);
    return hipGetLastError();
}

hipError_t launch_generic_gemm(int in_dtype, int dst_dtype, hipStream_t s, const GenArgs &a) {
    const dim3 grid((unsigned)((a.N + 31) / 32), (unsigned)((a.M + 31) / 32), (unsigned)a.batch), block(256);
#define FGE_GGK(InT, NarrowT, KT)                                                                      \
    do {                                                                                               \
        if (dst_dtype != FGE_F32) hipLaunchKernelGGL((generic_gemm_kernel<InT, NarrowT, KT>), grid, block, 0, s, a); \
        else                      hipLaunchKernelGGL((generic_gemm_kernel<InT, float, KT>), grid, block, 0, s, a);   \
    } while (0)
#define FGE_GG(InT, NarrowT)                                                                           \
    do {                                                                                               \
        if (a.K <= 32)      FGE_GGK(InT, NarrowT, 32);                                                 \
        else if (a.K <= 64) FGE_GGK(InT, NarrowT, 64);                                                 \
        else                FGE_GGK(InT, NarrowT, 128);                                                \
    } while (0)
    if (in_dtype == FGE_BF16)     FGE_GG(bf16_t, bf16_t);
    else if (in_dtype == FGE_F16) FGE_GG(f16_t, f16_t);
    else if (in_dtype == FGE_F8E4M3) FGE_GG(f8_t, bf16_t);
    else                          FGE_GG(float, bf16_t);
#undef FGE_GG
#undef FGE_GGK
    return hipGetLastError();
}

hipError_t launch_generic_act(int dtype, hipStream_t s, const GenArgs &a) {
    const int64_t total = (int64_t)a.batch * a.M * a.N;
    int64_t blocks = (total + 255) / 256;
    if (blocks > 256 * 32) blocks = 256 * 32;                           // grid-stride beyond that
    const dim3 grid((unsigned)blocks), block(256);
    if (dtype == FGE_BF16)     hipLaunchKernelGGL((generic_act_kernel<bf16_t>), grid, block, 0, s, a);
    else if (dtype == FGE_F16) hipLaunchKernelGGL((generic_act_kernel<f16_t>), grid, block, 0, s, a);
    else                       hipLaunchKernelGGL((generic_act_kernel<float>), grid, block, 0, s, a);
    return hipGetLastError();
}

// src is fp32 (the fused intermediate) or of the output type (the unfused A)
hipError_t launch_generic_row(int src_dtype, int out_dtype, hipStream_t s, const GenArgs &a) {
    const int64_t rows = (int64_t)a.batch * a.M;
    const dim3 grid((unsigned)((rows + 3) / 4)), block(256);
    if (src_dtype == FGE_F32 && a.X != a.dst && a.ldx % 4 == 0 && a.bsx % 4 == 0 && (reinterpret_cast<uintptr_t>(a.X) & 15) == 0 &&
        rows <= INT32_MAX) {
        // source rows on 16-byte boundaries: one workgroup per row; the row parked in LDS when it fits
        const dim3 g1((unsigned)rows);
        const size_t row_bytes = ((size_t)a.N * 4 + 15) / 16 * 16;
#define FGE_ROW(OT)                                                                                       \
        do {                                                                                               \
            if (row_bytes <= ((size_t)64 << 10) - 256)                                                     \
                hipLaunchKernelGGL((aligned_src_row_kernel<OT, true>), g1, block, row_bytes, s, a);        \
            else                                                                                           \
                hipLaunchKernelGGL((aligned_src_row_kernel<OT, false>), g1, block, 0, s, a);               \
        } while (0)
        if (out_dtype == FGE_BF16)     FGE_ROW(bf16_t);
        else if (out_dtype == FGE_F16) FGE_ROW(f16_t);
        else                           FGE_ROW(float);
#undef FGE_ROW
        return hipGetLastError();
    }
    // rows that registers hold: one wave per row of up to 512 (fp32: 256) columns, and of up to 2048 (1024) where there are enough rows for
    // that, else four - a workgroup of 256 per row, up to the 2^32 work items that the runtime launches.  Shorter rows, a few chunks of
    // 16 bytes, leave most of a wave idle there and go to the kernel with a value per lane (us, it -> so; bf16 259888 x 21 RMSNorm 47.6 -> 96.8,
    // 571 x 51 LayerNorm 2.5 -> 3.2, 300278 x 125 softmax 96.2 -> 133.6, f16 144010 x 153 softmax 59.9 -> 54.4, 75705 x 195 LayerNorm 38.0 -> 32.2;
    // fp32 146555 x 63 RMSNorm 29.1 -> 37.7, 827238 x 75 softmax 320.6 -> 258.0).  RMSNorm, whose values the other kernel reads
    // only twice, stays there longer (f16 195097 x 223 72.6 -> 89.8, bf16 211448 x 287 91.3 -> 99.7, fp32 997414 x 79 287.2 -> 326.6).
    const int per_wave = out_dtype == FGE_F32 ? 1024 : 2048;
    const bool rms = a.norm == FGE_NORM_RMSNORM;
    const int least = out_dtype == FGE_F32 ? (rms ? 96 : 64) : (rms ? 320 : 192);
    const bool one_wave = a.N <= per_wave / 4 || (rows >= 1024 && a.N <= per_wave);
    if (a.N > least && a.N <= 8192 && (one_wave || rows < (1 << 24)) && (src_dtype == FGE_F32 || src_dtype == out_dtype)) {
#define FGE_ANY_ROW(ST, OT, W, C) hipLaunchKernelGGL((any_row_kernel<ST, OT, W, C>), dim3((unsigned)(W == 1 ? (rows + 3) / 4 : rows)), block, 0, s, a)
#define FGE_ANY_ROWS(ST, OT)                                                                               \
        do {                                                                                               \
            constexpr int PER = 256 * Store<OT>::CW;                                                       \
            if (one_wave && a.N <= PER / 4)       FGE_ANY_ROW(ST, OT, 1, 1);                               \
            else if (one_wave && a.N <= PER / 2)  FGE_ANY_ROW(ST, OT, 1, 2);                               \
            else if (one_wave)                    FGE_ANY_ROW(ST, OT, 1, 4);                               \
            else if (a.N <= PER)                  FGE_ANY_ROW(ST, OT, 4, 1);                               \
            else if (a.N <= 2 * PER)              FGE_ANY_ROW(ST, OT, 4, 2);                               \
            else if (a.N <= 4 * PER)              FGE_ANY_ROW(ST, OT, 4, 4);                               \
            else if constexpr (sizeof(OT) == 4)   FGE_ANY_ROW(ST, OT, 4, 8);                               \
        } while (0)
        if (src_dtype == FGE_F32 && out_dtype == FGE_BF16)     FGE_ANY_ROWS(float, bf16_t);
        else if (src_dtype == FGE_F32 && out_dtype == FGE_F16) FGE_ANY_ROWS(float, f16_t);
        else if (src_dtype == FGE_F32)                         FGE_ANY_ROWS(float, float);
        else if (out_dtype == FGE_BF16)                        FGE_ANY_ROWS(bf16_t, bf16_t);
        else                                                   FGE_ANY_ROWS(f16_t, f16_t);
#undef FGE_ANY_ROWS
#undef FGE_ANY_ROW
        return hipGetLastError();
    }
    if (src_dtype == FGE_F32) {
        if (out_dtype == FGE_BF16)     hipLaunchKernelGGL((generic_row_kernel<float, bf16_t>), grid, block, 0, s, a);
        else if (out_dtype == FGE_F16) hipLaunchKernelGGL((generic_row_kernel<float, f16_t>), grid, block, 0, s, a);
        else                           hipLaunchKernelGGL((generic_row_kernel<float, float>), grid, block, 0, s, a);
    } else if (src_dtype == out_dtype) {
        if (out_dtype == FGE_BF16) hipLaunchKernelGGL((generic_row_kernel<bf16_t, bf16_t>), grid, block, 0, s, a);
        else                       hipLaunchKernelGGL((generic_row_kernel<f16_t, f16_t>), grid, block, 0, s, a);
    } else {
        return hipErrorInvalidValue;                                     // never asked for
    }
    return hipGetLastError();
}

}  // namespace fge
