// Forward of small batches by 64-sample columns, gfx950.
//
// A batch of a few columns (64-sample words) leaves the slab kernels mostly
// empty: a slab is 16 words wide whatever the batch, their blocks walk LDS
// tables and counter planes built for long runs of samples, and the four
// launches follow each other as latency chains of 4 to 6 us.  Here the packed
// tensors are laid out [W][rows], a column's rows contiguous, and a lane is a
// node (Sec. 3 "Nodes are parameterizations"; App. C.1 "Bit-packed
// inference"): a wave evaluates 64 nodes of one column or a few, so the work
// spreads over waves by nodes as well as by samples and no word is computed
// for padding.
//
//  k_col_encode  one wave per column and group of features, a lane a sample:
//                each wire's word is the ballot of its comparison (or of its
//                code bit), collected into lanes with v_writelane
//  k_col_layer   a lane gathers its node's K words of C columns from the L2
//                and folds them with the multiplexer tree
//  k_col_head    the last layer and the GroupSum counts of some classes for
//                one column: the column's input rows are staged in LDS, a
//                wave evaluates 64 nodes, the 64 x 64 transpose turns their
//                words into one word of node bits per sample, and each class
//                adds the popcount of its bits (Sec. 3 "Encoders and heads").
//                A block that holds every class also takes the argmax.
//  k_rows_argmax argmax of stored counts where the classes are spread over
//                several blocks
//
// What bounds them: launches and one or two memory latencies per kernel.
// Enqueued back to back from C, against the slab kernels on the same batch:
// 784 x 4 -> 4000 -> 4000, fan-in 4, 10 classes at 64 and 1024 samples 19.3 and
// 19.7 -> 13.0 us; 784 -> 1000 -> 1000, fan-in 6, at 4096 samples 18.8 -> 13.0;
// 784 x 7 -> 8000 -> 8000, fan-in 6, at 1024 31.9 -> 17.8; 9216 -> 32000 ->
// 32000, fan-in 6, at 64 78 -> 25 (37 with the slab's blocks on all XCDs).
#include "bl_device.h"

namespace bl {
namespace {

using dev::eval_node;
using dev::transpose64;
using dev::transpose_consts;

constexpr int kThreads = 256;
constexpr int kHeadThreads = 1024;
constexpr int kHeadWaves = kHeadThreads / kWave;
constexpr int kCntStride = kWave + 1;         // LDS words per class of counts

__device__ __forceinline__ uint32_t load_u32(const uint8_t *p)
{
    uint32_t v;
    __builtin_memcpy(&v, p, sizeof v);
    return v;
}

// Features of one wave: their wires fill a wave's lanes, whole dwords a row.
template <int B>
constexpr int col_features()
{
    return B == 1 ? 32 : B == 2 ? 32 : B <= 4 ? 16 : B == 5 ? 12 : 8;
}

template <int B, int KIND, int Q>
__device__ __forceinline__ void col_wires(const uint32_t (&px)[col_features<B>() / 4],
                                          uint32_t thv, uint32_t &lo, uint32_t &hi)
{
    constexpr int f = Q / B, t = Q % B;
    const uint32_t v = (px[f / 4] >> (8 * (f % 4))) & 0xFFu;
    uint64_t m;
    if constexpr (KIND == kEncThermometer) {
        m = __ballot(v > (uint32_t)__builtin_amdgcn_readlane((int)thv, Q));
    } else {
        // binary code: round(v (2^B - 1) / 255), no ties since 255 is odd
        const uint32_t code = (2u * v * ((1u << B) - 1u) + 255u) / 510u;
        m = __ballot((code >> t) & 1u);
    }
    lo = (uint32_t)bl_writelane((int)(uint32_t)m, Q, (int)lo);
    hi = (uint32_t)bl_writelane((int)(uint32_t)(m >> 32), Q, (int)hi);
    if constexpr (Q + 1 < col_features<B>() * B)
        col_wires<B, KIND, Q + 1>(px, thv, lo, hi);
}

template <int B, int KIND>
__global__ __launch_bounds__(kThreads) void k_col_encode(
    const uint8_t *__restrict__ x, int64_t n, int32_t d, const uint8_t *__restrict__ th,
    uint64_t *__restrict__ out, int32_t n_ftiles)
{
    constexpr int F = col_features<B>();
    const int lane = threadIdx.x % kWave;
    const int ft = blockIdx.x * (kThreads / kWave) +
                   __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if (ft >= n_ftiles)
        return;
    const int64_t col = blockIdx.y;
    // the last group starts earlier and repeats features that it does not write
    const int f0 = max(min(ft * F, d - F), 0);
    const int skip = ft * F - f0;
    const int nf = min(F, d - f0);
    const int64_t s = col * kWave + lane;
    uint32_t px[F / 4];
    const uint8_t *row = x + min(s, n - 1) * d + f0;
    if (nf == F) {
#pragma unroll
        for (int q = 0; q < F / 4; ++q)
            px[q] = load_u32(row + 4 * q);
    } else {
#pragma unroll
        for (int q = 0; q < F / 4; ++q) {
            px[q] = 0;
            for (int u = 0; u < 4; ++u)
                if (4 * q + u < nf)
                    px[q] |= (uint32_t)row[4 * q + u] << (8 * u);
        }
    }
    uint32_t thv = 255;                        // nothing is above 255
    if (KIND == kEncThermometer && lane < nf * B)
        thv = th[(int64_t)f0 * B + lane];
#pragma unroll
    for (int q = 0; q < F / 4; ++q)
        px[q] = s < n ? px[q] : 0u;            // padding samples encode to 0
    uint32_t lo = 0, hi = 0;
    col_wires<B, KIND, 0>(px, thv, lo, hi);
    if (lane >= skip * B && lane < nf * B)
        out[col * ((int64_t)d * B) + (int64_t)f0 * B + lane] = (uint64_t)hi << 32 | lo;
}

template <int K, int C>
__global__ __launch_bounds__(kThreads) void k_col_layer(
    const uint64_t *__restrict__ in, int32_t w_in, const int32_t *__restrict__ conn,
    const uint64_t *__restrict__ tables, int32_t w_out, uint64_t *__restrict__ out, int32_t W,
    int32_t n_cg)
{
    // column groups vary fastest, so that blocks of one group tend to share
    // an XCD and its L2
    const int cg = blockIdx.x % n_cg;
    const int j = (blockIdx.x / n_cg) * kThreads + threadIdx.x;
    const int jc = min(j, w_out - 1);
    int32_t idx[K];
#pragma unroll
    for (int i = 0; i < K; ++i)
        idx[i] = conn[(int64_t)jc * K + i];
    const uint64_t T = tables[jc];
    uint32_t xv[2 * C][K], o[2 * C];
#pragma unroll
    for (int r = 0; r < C; ++r) {
        const uint64_t *src = in + (int64_t)min(cg * C + r, W - 1) * w_in;
#pragma unroll
        for (int i = 0; i < K; ++i) {
            const uint64_t v = src[idx[i]];
            xv[2 * r][i] = (uint32_t)v;
            xv[2 * r + 1][i] = (uint32_t)(v >> 32);
        }
    }
    eval_node<K, C>(T, xv, o);
#pragma unroll
    for (int r = 0; r < C; ++r)
        if (j < w_out && cg * C + r < W)
            out[(int64_t)(cg * C + r) * w_out + j] = (uint64_t)o[2 * r + 1] << 32 | o[2 * r];
}

// One block: the classes [c0, c0 + cpb) of column blockIdx.x.  LDS: the
// column's w_in words (STAGED), then the classes' counts, kCntStride words
// each, then the argmax partials.
template <int K, bool STAGED>
__global__ __launch_bounds__(kHeadThreads) void k_col_head(
    const uint64_t *__restrict__ in, int32_t w_in, const int32_t *__restrict__ conn,
    const uint64_t *__restrict__ tables, int32_t g, int32_t c, int32_t cpb, int64_t n,
    int32_t *__restrict__ counts, int32_t *__restrict__ argmax)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    uint64_t *s_in = reinterpret_cast<uint64_t *>(smem);
    int32_t *s_cnt = reinterpret_cast<int32_t *>(smem + (STAGED ? (size_t)(w_in + 1) / 2 * 16 : 0));
    const int tid = threadIdx.x;
    const int lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int64_t col = blockIdx.x;
    const int c0 = blockIdx.y * cpb;
    const int nc = min(cpb, c - c0);
    const int n0 = c0 * g, n1 = n0 + nc * g;
    const uint64_t *src = in + col * w_in;

    // the wave's first nodes, requested before the rows are staged
    int32_t idx[K];
    uint64_t T = 0;
    auto fetch = [&](int base) {
        const int j = min(base + lane, n1 - 1);
#pragma unroll
        for (int i = 0; i < K; ++i)
            idx[i] = conn[(int64_t)j * K + i];
        T = tables[j];
    };
    int base = n0 + wave * kWave;
    if (base < n1)
        fetch(base);
    if constexpr (STAGED) {
        for (int e = tid; e < w_in / 2; e += kHeadThreads) {
            u32x4 v;
            __builtin_memcpy(&v, src + 2 * e, sizeof v);
            reinterpret_cast<u32x4 *>(s_in)[e] = v;
        }
        if (w_in % 2 != 0 && tid == 0)
            s_in[w_in - 1] = src[w_in - 1];
    }
    for (int e = tid; e < nc * kCntStride; e += kHeadThreads)
        s_cnt[e] = 0;
    __syncthreads();

    const dev::Transpose tr = transpose_consts(lane);
    while (base < n1) {
        uint32_t xv[2][K], o[2];
#pragma unroll
        for (int i = 0; i < K; ++i) {
            const uint64_t v = STAGED ? s_in[idx[i]] : src[idx[i]];
            xv[0][i] = (uint32_t)v;
            xv[1][i] = (uint32_t)(v >> 32);
        }
        const uint64_t Tc = T;
        const int next = base + kHeadThreads;
        if (next < n1)
            fetch(next);
        eval_node<K, 1>(Tc, xv, o);
        // lane = node -> lane = sample, bit l = node base + l
        transpose64(o[0], o[1], tr);
        const uint64_t bits = (uint64_t)o[1] << 32 | o[0];
        const int end = min(base + kWave, n1);
        for (int cls = base / g; cls * g < end; ++cls) {
            const int a = max(cls * g, base) - base, b = min((cls + 1) * g, end) - base;
            const uint64_t m = (~0ull >> (kWave - (b - a))) << a;
            atomicAdd(&s_cnt[(cls - c0) * kCntStride + lane], (int32_t)__popcll(bits & m));
        }
        base = next;
    }
    __syncthreads();

    const int64_t s0 = col * kWave;
    const int rows = (int)min((int64_t)kWave, n - s0);
    if (counts)
        for (int e = tid; e < rows * nc; e += kHeadThreads) {
            const int r = e / nc, k = e - r * nc;
            counts[(s0 + r) * c + c0 + k] = s_cnt[k * kCntStride + r];
        }
    if (argmax) {
        // every class is here: each wave scans a run of them in order, and
        // wave 0 merges the runs (largest count, lowest class on ties)
        int32_t *s_best = s_cnt + nc * kCntStride, *s_at = s_best + kHeadWaves * kWave;
        const int per = (c + kHeadWaves - 1) / kHeadWaves;
        int32_t best = -1, at = 0;
        for (int k = wave * per; k < min((wave + 1) * per, c); ++k) {
            const int32_t v = s_cnt[k * kCntStride + lane];
            if (v > best) {
                best = v;
                at = k;
            }
        }
        s_best[wave * kWave + lane] = best;
        s_at[wave * kWave + lane] = at;
        __syncthreads();
        if (wave == 0 && lane < rows) {
            for (int w = 1; w < kHeadWaves; ++w)
                if (s_best[w * kWave + lane] > best) {
                    best = s_best[w * kWave + lane];
                    at = s_at[w * kWave + lane];
                }
            argmax[s0 + lane] = at;
        }
    }
}

__global__ __launch_bounds__(kThreads) void k_rows_argmax(const int32_t *__restrict__ counts,
                                                          int64_t n, int32_t c,
                                                          int32_t *__restrict__ argmax)
{
    const int64_t s = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (s >= n)
        return;
    int32_t best = -1, at = 0;
#pragma unroll 4
    for (int k = 0; k < c; ++k) {
        const int32_t v = counts[s * c + k];
        if (v > best) {
            best = v;
            at = k;
        }
    }
    argmax[s] = at;
}

template <int B>
hipError_t launch_encode_b(const uint8_t *x, int64_t n, int32_t d, const uint8_t *th,
                           uint64_t *out, int kind, hipStream_t stream)
{
    constexpr int F = col_features<B>();
    const int32_t n_ftiles = (d + F - 1) / F;
    const unsigned W = (unsigned)((n + 63) / 64);
    const dim3 grid((n_ftiles + kThreads / kWave - 1) / (kThreads / kWave), W);
    if (kind == kEncThermometer)
        hipLaunchKernelGGL((k_col_encode<B, kEncThermometer>), grid, dim3(kThreads), 0, stream, x,
                           n, d, th, out, n_ftiles);
    else
        hipLaunchKernelGGL((k_col_encode<B, kEncBinary>), grid, dim3(kThreads), 0, stream, x, n, d,
                           th, out, n_ftiles);
    return hipGetLastError();
}

template <int K, int C>
hipError_t launch_layer_kc(const uint64_t *in, int32_t w_in, const int32_t *conn,
                           const uint64_t *tables, int32_t w_out, uint64_t *out, int32_t W,
                           hipStream_t stream)
{
    const int32_t n_cg = (W + C - 1) / C;
    const int64_t blocks = (int64_t)n_cg * ((w_out + kThreads - 1) / kThreads);
    if (blocks > 0x7fffffff)
        return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((k_col_layer<K, C>), dim3((unsigned)blocks), dim3(kThreads), 0, stream, in,
                       w_in, conn, tables, w_out, out, W, n_cg);
    return hipGetLastError();
}

template <int K>
hipError_t launch_layer_k(const uint64_t *in, int32_t w_in, const int32_t *conn,
                          const uint64_t *tables, int32_t w_out, uint64_t *out, int32_t W,
                          hipStream_t stream)
{
    // a lane serves 4 or 2 columns of its node once that still leaves a wave
    // per SIMD: the table's masks are then extracted once for all of them
    const int64_t waves = (int64_t)W * ((w_out + kWave - 1) / kWave);
    if (waves >= 4 * 2048 && W >= 4)
        return launch_layer_kc<K, 4>(in, w_in, conn, tables, w_out, out, W, stream);
    if (waves >= 2 * 2048 && W >= 2)
        return launch_layer_kc<K, 2>(in, w_in, conn, tables, w_out, out, W, stream);
    return launch_layer_kc<K, 1>(in, w_in, conn, tables, w_out, out, W, stream);
}

template <int K>
hipError_t launch_head_k(const uint64_t *in, int32_t w_in, const int32_t *conn,
                         const uint64_t *tables, int32_t g, int32_t c, int64_t n,
                         const ColumnHeadPlan &hp, int32_t *counts, int32_t *argmax,
                         hipStream_t stream)
{
    const dim3 grid((unsigned)((n + 63) / 64), (unsigned)hp.splits);
    int32_t *am = hp.splits == 1 ? argmax : nullptr;
    if (hp.staged)
        hipLaunchKernelGGL((k_col_head<K, true>), grid, dim3(kHeadThreads), hp.lds, stream, in,
                           w_in, conn, tables, g, c, hp.cpb, n, counts, am);
    else
        hipLaunchKernelGGL((k_col_head<K, false>), grid, dim3(kHeadThreads), hp.lds, stream, in,
                           w_in, conn, tables, g, c, hp.cpb, n, counts, am);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || hp.splits == 1 || !argmax)
        return e;
    hipLaunchKernelGGL(k_rows_argmax, dim3((unsigned)((n + kThreads - 1) / kThreads)),
                       dim3(kThreads), 0, stream, counts, n, c, argmax);
    return hipGetLastError();
}

}  // namespace

// A head block's rounds of 16 waves of 64 nodes before its classes are spread
// over more blocks.  4 against 2 and 8: 4000 nodes of fan-in 4 (4 rounds in one
// block, no argmax launch) 11.6 against 14.1 us, 32000 of fan-in 6 34.0 against
// 34.5 and 41.8 us at 1024 samples; 8000 of fan-in 6 17.6 against 14.2 and 23.1.
constexpr int kHeadRounds = 4;

ColumnHeadPlan plan_column_head(int32_t w_in, int32_t w_out, int32_t c)
{
    ColumnHeadPlan p{};
    const int32_t g = w_out / c;
    // classes per block: all of them, or as many as keep a block to
    // kHeadRounds rounds
    const int64_t per_block = (int64_t)kHeadRounds * kHeadThreads;
    int32_t cpb = (int32_t)(per_block / g);
    cpb = cpb < 1 ? 1 : cpb > c ? c : cpb;
    p.splits = (c + cpb - 1) / cpb;
    p.cpb = (c + p.splits - 1) / p.splits;
    p.splits = (c + p.cpb - 1) / p.cpb;
    const size_t cnt = (size_t)p.cpb * kCntStride * 4 + 2 * kHeadWaves * kWave * 4;
    const size_t rows = (size_t)(w_in + 1) / 2 * 16;
    p.staged = cnt + rows <= kColumnLds;
    p.lds = cnt + (p.staged ? rows : 0);
    p.ok = p.lds <= kColumnLds;
    return p;
}

hipError_t launch_column_encode(const uint8_t *x, int64_t n, int32_t d, const uint8_t *th,
                                int32_t b, uint64_t *out, int kind, hipStream_t stream)
{
    switch (b) {
    case 1: return launch_encode_b<1>(x, n, d, th, out, kind, stream);
    case 2: return launch_encode_b<2>(x, n, d, th, out, kind, stream);
    case 3: return launch_encode_b<3>(x, n, d, th, out, kind, stream);
    case 4: return launch_encode_b<4>(x, n, d, th, out, kind, stream);
    case 5: return launch_encode_b<5>(x, n, d, th, out, kind, stream);
    case 6: return launch_encode_b<6>(x, n, d, th, out, kind, stream);
    case 7: return launch_encode_b<7>(x, n, d, th, out, kind, stream);
    case 8: return launch_encode_b<8>(x, n, d, th, out, kind, stream);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_column_layer(const uint64_t *in, int32_t w_in, int32_t W, const int32_t *conn,
                               const uint64_t *tables, int32_t w_out, int32_t k, uint64_t *out,
                               hipStream_t stream)
{
    switch (k) {
    case 1: return launch_layer_k<1>(in, w_in, conn, tables, w_out, out, W, stream);
    case 2: return launch_layer_k<2>(in, w_in, conn, tables, w_out, out, W, stream);
    case 3: return launch_layer_k<3>(in, w_in, conn, tables, w_out, out, W, stream);
    case 4: return launch_layer_k<4>(in, w_in, conn, tables, w_out, out, W, stream);
    case 5: return launch_layer_k<5>(in, w_in, conn, tables, w_out, out, W, stream);
    case 6: return launch_layer_k<6>(in, w_in, conn, tables, w_out, out, W, stream);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_column_head(const uint64_t *in, int32_t w_in, const int32_t *conn,
                              const uint64_t *tables, int32_t w_out, int32_t k, int32_t c,
                              int64_t n, const ColumnHeadPlan &hp, int32_t *counts,
                              int32_t *argmax, hipStream_t stream)
{
    const int32_t g = w_out / c;
    switch (k) {
    case 1: return launch_head_k<1>(in, w_in, conn, tables, g, c, n, hp, counts, argmax, stream);
    case 2: return launch_head_k<2>(in, w_in, conn, tables, g, c, n, hp, counts, argmax, stream);
    case 3: return launch_head_k<3>(in, w_in, conn, tables, g, c, n, hp, counts, argmax, stream);
    case 4: return launch_head_k<4>(in, w_in, conn, tables, g, c, n, hp, counts, argmax, stream);
    case 5: return launch_head_k<5>(in, w_in, conn, tables, g, c, n, hp, counts, argmax, stream);
    case 6: return launch_head_k<6>(in, w_in, conn, tables, g, c, n, hp, counts, argmax, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace bl
