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
//                the rows and the transpose of the large encoder, without its
//                tiles
//  k_col_layer   a lane gathers its node's K words of C columns from the L2
//                and folds them with the multiplexer tree
//  k_col_head    the last layer and the GroupSum counts of some classes for
//                one column: the column's input rows are staged in LDS, a
//                wave evaluates 64 nodes, the 64 x 64 transpose turns their
//                words into one word of node bits per sample, and each class
//                adds the popcount of its bits (Sec. 3 "Encoders and heads").
//                A block that holds every class also takes the argmax.
//  k_col_network all of it in one block and launch, where a column is little work
//  k_rows_argmax argmax of stored counts where the classes are spread over
//                several blocks
//
// What bounds them: launches and one or two memory latencies per kernel.
// Enqueued back to back from C, against the slab kernels on the same batch:
// 784 x 4 -> 4000 -> 4000, fan-in 4, 10 classes at 64 and 1024 samples 19.3 and
// 19.7 -> 13.0 us; 784 -> 1000 -> 1000, fan-in 6, at 4096 samples 18.8 -> 13.0;
// 784 x 7 -> 8000 -> 8000, fan-in 6, at 1024 31.9 -> 17.8; 9216 -> 32000 ->
// 32000, fan-in 6, at 64 78 -> 25 (37 with the slab's blocks on all XCDs).
#include <type_traits>

#include "bl_device.h"
#include "encode_row.h"

namespace bl {
namespace {

using namespace dev;

constexpr int kThreads = 256;
constexpr int kHeadThreads = 1024;
constexpr int kHeadWaves = kHeadThreads / kWave;
constexpr int kCntStride = kWave + 1;         // LDS words per class of counts

// A node of a layer with a fan-in array, whose output its first kp slots give
// whatever the others hold: the others read wire 0 and the table, repeated over
// them, ignores them, so that nodes of all fan-ins run as nodes of K inputs.
// kp >= K changes nothing.
template <int K>
__device__ __forceinline__ void keep_slots(int kp, int32_t *idx, uint64_t &T)
{
#pragma unroll
    for (int i = 0; i < K; ++i) {
        const uint64_t low = (1ull << (1 << i)) - 1;
        T = i < kp ? T : (T & low) | T << (1 << i);
        idx[i] = i < kp ? idx[i] : 0;
    }
}

// One wave's group of features of one column: their pixels (a lane a sample)
// and, in lane k < kS, the thresholds of slot k.
template <int B>
struct ColGroup {
    using G = EncGeom<B, 1>;
    uint32_t px[G::kQ], th4;
    int f0, skip, nf;

    // group ft of n_ftiles; the last one starts earlier and repeats features
    // that it does not write
    __device__ __forceinline__ void load(const uint8_t *__restrict__ x, int64_t n, int32_t d,
                                         const uint8_t *__restrict__ th, int kind, int64_t col,
                                         int ft)
    {
        const int lane = threadIdx.x % kWave;
        f0 = max(min(ft * G::kFPG, d - G::kFPG), 0);
        skip = ft * G::kFPG - f0;
        nf = min(G::kFPG, d - f0);
        const uint8_t *row = x + min(col * kWave + lane, n - 1) * d + f0;
        if (nf == G::kFPG) {
#pragma unroll
            for (int q = 0; q < G::kQ; ++q)
                px[q] = load_u32(row + 4 * q);
        } else {
#pragma unroll
            for (int q = 0; q < G::kQ; ++q) {
                px[q] = 0;
                for (int u = 0; u < 4; ++u)
                    if (4 * q + u < nf)
                        px[q] |= (uint32_t)row[4 * q + u] << (8 * u);
            }
        }
        th4 = ~0u;
        if (kind == kEncThermometer && lane < G::kS) {
            const int f = lane / B * 4, t = lane % B;
            th4 = 0;
#pragma unroll
            for (int u = 0; u < 4; ++u)
                th4 |= (f + u < nf ? (uint32_t)th[(int64_t)(f0 + f + u) * B + t] : 255u)
                       << (8 * u);
        }
    }

    // the group's words: lane p returns the one of wire row_wire(p), at wire
    // f0 * B + row_wire(p) of the tensor where `mine`
    __device__ __forceinline__ uint64_t words(int64_t n, int kind, int64_t col, const Transpose &tr,
                                              const uint32_t (&mk)[8], int wire, bool &mine)
    {
        const bool in = col * kWave + threadIdx.x % kWave < n;
#pragma unroll
        for (int q = 0; q < G::kQ; ++q)
            px[q] = in ? px[q] : 0u;               // padding samples encode to 0
        uint32_t lo, hi;
        if (kind == kEncThermometer) {
            uint32_t nt[16];
#pragma unroll
            for (int k = 0; k < G::kS; ++k)
                nt[k] = ~(uint32_t)__builtin_amdgcn_readlane((int)th4, k);
            row_thermometer<B>(px, nt, mk, lo, hi);
        } else {
            row_binary<B>(px, mk, lo, hi);
        }
        transpose64(lo, hi, tr);
        mine = wire >= skip * B && wire < nf * B;
        return (uint64_t)hi << 32 | lo;
    }
};

template <int B>
__global__ __launch_bounds__(kThreads) void k_col_encode(
    const uint8_t *__restrict__ x, int64_t n, int32_t d, const uint8_t *__restrict__ th,
    uint64_t *__restrict__ out, int32_t n_ftiles, int kind)
{
    const int lane = threadIdx.x % kWave;
    const int ft = blockIdx.x * (kThreads / kWave) +
                   __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if (ft >= n_ftiles)
        return;
    const int64_t col = blockIdx.y;
    ColGroup<B> g;
    g.load(x, n, d, th, kind, col, ft);
    const Transpose tr = transpose_consts(lane);
    uint32_t mk[8];
    row_masks(mk);
    const int wire = row_wire<B>(lane);
    bool mine;
    const uint64_t w = g.words(n, kind, col, tr, mk, wire, mine);
    if (mine)
        out[col * ((int64_t)d * B) + (int64_t)g.f0 * B + wire] = w;
}

template <int K, int C>
__global__ __launch_bounds__(kThreads) void k_col_layer(
    const uint64_t *__restrict__ in, int32_t w_in, const int32_t *__restrict__ conn,
    const uint64_t *__restrict__ tables, int32_t w_out, uint64_t *__restrict__ out, int32_t W,
    int32_t n_cg, const uint8_t *__restrict__ fanin)
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
    uint64_t T = tables[jc];
    if (fanin)
        keep_slots<K>(fanin[jc / kSpecPass], idx, T);
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

// A block's counts (LDS, nc classes from c0, kCntStride words each) of column col
// to counts [n][c] and, where the block holds every class, to argmax; all
// threads, after a barrier.
__device__ __forceinline__ void column_results(int32_t *s_cnt, int64_t col, int64_t n, int32_t c,
                                               int c0, int nc, int32_t *__restrict__ counts,
                                               int32_t *__restrict__ argmax)
{
    const int tid = threadIdx.x;
    const int lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
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

// Adds the popcounts of a wave's 64 node words (lane = node base + lane; lanes past
// n1 hold any words, which the masks leave out) to the counts of their classes.
__device__ __forceinline__ void count_nodes(uint32_t (&o)[2], int base, int n1, int g, int c0,
                                            const Transpose &tr, int32_t *s_cnt)
{
    const int lane = threadIdx.x % kWave;
    // lane = node -> lane = sample, bit l = node base + l
    transpose64(o[0], o[1], tr);
    const uint64_t bits = (uint64_t)o[1] << 32 | o[0];
    const int end = min(base + kWave, n1);
    for (int cls = base / g; cls * g < end; ++cls) {
        const int a = max(cls * g, base) - base, b = min((cls + 1) * g, end) - base;
        const uint64_t m = (~0ull >> (kWave - (b - a))) << a;
        atomicAdd(&s_cnt[(cls - c0) * kCntStride + lane], (int32_t)__popcll(bits & m));
    }
}

// One block: the classes [c0, c0 + cpb) of column blockIdx.x.  LDS: the
// column's w_in words (STAGED), then the classes' counts, kCntStride words
// each, then the argmax partials.
template <int K, bool STAGED>
__global__ __launch_bounds__(kHeadThreads) void k_col_head(
    const uint64_t *__restrict__ in, int32_t w_in, const int32_t *__restrict__ conn,
    const uint64_t *__restrict__ tables, int32_t g, int32_t c, int32_t cpb, int64_t n,
    int32_t *__restrict__ counts, int32_t *__restrict__ argmax,
    const uint8_t *__restrict__ fanin)
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
    int kp = K;
    auto fetch = [&](int base) {
        const int j = min(base + lane, n1 - 1);
#pragma unroll
        for (int i = 0; i < K; ++i)
            idx[i] = conn[(int64_t)j * K + i];
        T = tables[j];
        if (fanin)
            kp = fanin[j / kSpecPass];
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
        if (fanin)
            keep_slots<K>(kp, idx, T);
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
        count_nodes(o, base, n1, g, c0, tr, s_cnt);
        base = next;
    }
    __syncthreads();

    column_results(s_cnt, col, n, c, c0, nc, counts, argmax);
}

// A lane's node of K inputs on one column (s_in: the column's words).
template <int K>
__device__ __forceinline__ void eval_lds(const uint64_t *s_in, const int32_t (&idx)[6], uint64_t T,
                                         uint32_t (&o)[2])
{
    uint32_t xv[2][K];
#pragma unroll
    for (int i = 0; i < K; ++i) {
        const uint64_t v = s_in[idx[i]];
        xv[0][i] = (uint32_t)v;
        xv[1][i] = (uint32_t)(v >> 32);
    }
    eval_node<K, 1>(T, xv, o);
}

// The whole network of one column in one block: wires, hidden layers and counts
// in LDS (two buffers of rows_a and rows_b words, used in turn, then the counts
// and argmax partials).  SPEC: some layer has a fan-in array (tested per layer
// in the plain kernel it cost 0.2 of the 9.9 us of 784 -> 1000 -> 1000).
template <int B, bool SPEC>
__global__ __launch_bounds__(kHeadThreads) void k_col_network(
    const uint8_t *__restrict__ x, int64_t n, int32_t d, const uint8_t *__restrict__ th, int kind,
    int32_t n_ftiles, ColumnNetwork net, int32_t rows_a, int32_t rows_b, int32_t c,
    int32_t *__restrict__ counts, int32_t *__restrict__ argmax)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    uint64_t *buf[2] = {reinterpret_cast<uint64_t *>(smem),
                        reinterpret_cast<uint64_t *>(smem) + rows_a};
    int32_t *s_cnt = reinterpret_cast<int32_t *>(buf[1] + rows_b);
    const int tid = threadIdx.x;
    const int lane = tid % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int64_t col = blockIdx.x;
    const Transpose tr = transpose_consts(lane);

    // the next nodes' connections and tables, always one task ahead
    int32_t idx[6];
    uint64_t T = 0;
    int kp = 6;
    auto fetch = [&](int l, int base) {
        const int k = net.k[l], j = min(base + lane, net.w[l] - 1);
        const int32_t *src = net.conn[l] + (int64_t)j * k;
        // whole-vector loads: a dword at a time they were most of the kernel
        switch (k) {
        case 1: __builtin_memcpy(idx, src, 4); break;
        case 2: __builtin_memcpy(idx, src, 8); break;
        case 3: __builtin_memcpy(idx, src, 12); break;
        case 4: __builtin_memcpy(idx, src, 16); break;
        case 5: __builtin_memcpy(idx, src, 20); break;
        default: __builtin_memcpy(idx, src, 24); break;
        }
        T = net.tables[l][j];
        if (SPEC && net.fanin[l])
            kp = net.fanin[l][j / kSpecPass];
    };
    if (wave < n_ftiles) {
        ColGroup<B> cur, next;
        cur.load(x, n, d, th, kind, col, wave);
        uint32_t mk[8];
        row_masks(mk);
        const int wire = row_wire<B>(lane);
        for (int ft = wave; ft < n_ftiles; ft += kHeadWaves) {
            if (ft + kHeadWaves < n_ftiles)
                next.load(x, n, d, th, kind, col, ft + kHeadWaves);
            else
                fetch(0, wave * kWave);
            bool mine;
            const uint64_t w = cur.words(n, kind, col, tr, mk, wire, mine);
            if (mine)
                buf[0][cur.f0 * B + wire] = w;
            cur = next;
        }
    } else {
        fetch(0, wave * kWave);
    }
    for (int e = tid; e < c * kCntStride; e += kHeadThreads)
        s_cnt[e] = 0;
    __syncthreads();

    for (int l = 0; l < net.n_layers; ++l) {
        const bool last = l == net.n_layers - 1;
        const int w = net.w[l], k = net.k[l];
        const uint64_t *s_in = buf[l % 2];
        uint64_t *s_out = buf[(l + 1) % 2];
        if (wave * kWave >= w && !last)
            fetch(l + 1, wave * kWave);
        for (int base = wave * kWave; base < w; base += kHeadThreads) {
            int32_t at[6];
#pragma unroll
            for (int i = 0; i < 6; ++i)
                at[i] = idx[i];
            uint64_t Tc = T;
            if (SPEC && net.fanin[l])
                keep_slots<6>(kp, at, Tc);
            if (base + kHeadThreads < w)
                fetch(l, base + kHeadThreads);
            else if (!last)
                fetch(l + 1, wave * kWave);
            uint32_t o[2];
            switch (k) {
            case 1: eval_lds<1>(s_in, at, Tc, o); break;
            case 2: eval_lds<2>(s_in, at, Tc, o); break;
            case 3: eval_lds<3>(s_in, at, Tc, o); break;
            case 4: eval_lds<4>(s_in, at, Tc, o); break;
            case 5: eval_lds<5>(s_in, at, Tc, o); break;
            default: eval_lds<6>(s_in, at, Tc, o); break;
            }
            if (last)
                count_nodes(o, base, w, w / c, 0, tr, s_cnt);
            else if (base + lane < w)
                s_out[base + lane] = (uint64_t)o[1] << 32 | o[0];
        }
        __syncthreads();
    }
    column_results(s_cnt, col, n, c, 0, c, counts, argmax);
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
    constexpr int F = EncGeom<B, 1>::kFPG;
    const int32_t n_ftiles = (d + F - 1) / F;
    const unsigned W = (unsigned)((n + 63) / 64);
    const dim3 grid((n_ftiles + kThreads / kWave - 1) / (kThreads / kWave), W);
    hipLaunchKernelGGL(k_col_encode<B>, grid, dim3(kThreads), 0, stream, x, n, d, th, out,
                       n_ftiles, kind);
    return hipGetLastError();
}

template <int B>
hipError_t launch_network_b(const uint8_t *x, int64_t n, int32_t d, const uint8_t *th, int kind,
                            const ColumnNetwork &net, int32_t c, int32_t *counts, int32_t *argmax,
                            hipStream_t stream)
{
    constexpr int F = EncGeom<B, 1>::kFPG;
    bool spec = false;
    for (int32_t l = 0; l < net.n_layers; ++l)
        spec = spec || net.fanin[l];
    const auto kernel = spec ? k_col_network<B, true> : k_col_network<B, false>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)((n + 63) / 64)), dim3(kHeadThreads), net.lds,
                       stream, x, n, d, th, kind, (d + F - 1) / F, net, net.rows_a, net.rows_b, c,
                       counts, argmax);
    return hipGetLastError();
}

template <int K, int C>
hipError_t launch_layer_kc(const uint64_t *in, int32_t w_in, const int32_t *conn,
                           const uint64_t *tables, int32_t w_out, uint64_t *out, int32_t W,
                           const uint8_t *fanin, hipStream_t stream)
{
    const int32_t n_cg = (W + C - 1) / C;
    const int64_t blocks = (int64_t)n_cg * ((w_out + kThreads - 1) / kThreads);
    if (blocks > 0x7fffffff)
        return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((k_col_layer<K, C>), dim3((unsigned)blocks), dim3(kThreads), 0, stream, in,
                       w_in, conn, tables, w_out, out, W, n_cg, fanin);
    return hipGetLastError();
}

template <int K>
hipError_t launch_layer_k(const uint64_t *in, int32_t w_in, const int32_t *conn,
                          const uint64_t *tables, int32_t w_out, uint64_t *out, int32_t W,
                          const uint8_t *fanin, hipStream_t stream)
{
    // a lane serves 4 or 2 columns of its node once that still leaves a wave
    // per SIMD: the table's masks are then extracted once for all of them
    const int64_t waves = (int64_t)W * ((w_out + kWave - 1) / kWave);
    if (waves >= 4 * 2048 && W >= 4)
        return launch_layer_kc<K, 4>(in, w_in, conn, tables, w_out, out, W, fanin, stream);
    if (waves >= 2 * 2048 && W >= 2)
        return launch_layer_kc<K, 2>(in, w_in, conn, tables, w_out, out, W, fanin, stream);
    return launch_layer_kc<K, 1>(in, w_in, conn, tables, w_out, out, W, fanin, stream);
}

template <int K>
hipError_t launch_head_k(const uint64_t *in, int32_t w_in, const int32_t *conn,
                         const uint64_t *tables, int32_t g, int32_t c, int64_t n,
                         const ColumnHeadPlan &hp, int32_t *counts, int32_t *argmax,
                         const uint8_t *fanin, hipStream_t stream)
{
    const dim3 grid((unsigned)((n + 63) / 64), (unsigned)hp.splits);
    int32_t *am = hp.splits == 1 ? argmax : nullptr;
    if (hp.staged)
        hipLaunchKernelGGL((k_col_head<K, true>), grid, dim3(kHeadThreads), hp.lds, stream, in,
                           w_in, conn, tables, g, c, hp.cpb, n, counts, am, fanin);
    else
        hipLaunchKernelGGL((k_col_head<K, false>), grid, dim3(kHeadThreads), hp.lds, stream, in,
                           w_in, conn, tables, g, c, hp.cpb, n, counts, am, fanin);
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
    const size_t rows = ((size_t)w_in + 1) / 2 * 16;
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

// The most wave instructions of a column that one block runs.  Its launch saves
// the host two others and the GPU their gaps, but one CU does the column's work:
// 784 -> 1000 -> 1000 at fan-in 6 (10330) 10.3 us against 13.0 for the stage
// kernels at 64 to 4096 samples, 10.5 against 15.1 at 16384; 784 x 3 -> 2500 ->
// 2516 at fan-in 5 (16810) 14.3 against 13.2, 784 x 4 -> 4000 -> 4000 at fan-in 4
// (20230) 15.8 against 13.1.
constexpr int64_t kNetworkMaxWork = 14000;
// The most columns: three rounds of blocks, one a CU, of 3 to 8 us each, or two
// where rows are shorter than a group of features and are loaded a byte at a
// time.  Against the stage kernels and the slab kernels at 512 columns 784 -> 100
// -> 100 at fan-in 4 13.4 : 16.1 : 20.8 us, 32 -> 16 -> 16 14.1 : 12.1 : 14.7; at
// 768 19.8 : 21.8 : 22.9 and 20.0 : 12.4 : 14.7; at 1024 26.6 : 26.1 : 27.2.
constexpr int64_t kNetworkMaxColumns = 768;
constexpr int64_t kNetworkMaxColumnsShortRows = 512;
ColumnNetwork plan_column_network(int32_t d, int32_t b, const int32_t *w, const int32_t *k,
                                  int32_t n_layers, int32_t c, int64_t n)
{
    ColumnNetwork net{};
    if (n_layers > kColumnMaxLayers)
        return net;
    int32_t rows[2] = {d * b, 0};
    // wave instructions of a column: a group of 64 wires, 64 nodes, 64 nodes counted
    int64_t work = ((int64_t)d * b + 63) / 64 * 130;
    for (int32_t l = 0; l < n_layers; ++l) {
        net.w[l] = w[l];
        net.k[l] = k[l];
        const int64_t chunks = (w[l] + kWave - 1) / kWave;
        work += chunks * (k[l] <= 4 ? 70 : k[l] == 5 ? 110 : 230);
        if (l == n_layers - 1)
            work += chunks * 80;
        else
            rows[(l + 1) % 2] = rows[(l + 1) % 2] > w[l] ? rows[(l + 1) % 2] : w[l];
    }
    net.n_layers = n_layers;
    net.rows_a = rows[0];
    net.rows_b = rows[1];
    net.lds = ((size_t)rows[0] + rows[1]) * 8 + (size_t)c * kCntStride * 4 +
              2 * kHeadWaves * kWave * 4;
    const int64_t most = d < 4 * group_quads(b) ? kNetworkMaxColumnsShortRows
                                                : kNetworkMaxColumns;
    net.ok = net.lds <= kColumnLds && work <= kNetworkMaxWork && n <= kWave * most;
    return net;
}

hipError_t launch_column_network(const uint8_t *x, int64_t n, int32_t d, const uint8_t *th,
                                 int32_t b, int kind, const ColumnNetwork &net, int32_t c,
                                 int32_t *counts, int32_t *argmax, hipStream_t stream)
{
    switch (b) {
    case 1: return launch_network_b<1>(x, n, d, th, kind, net, c, counts, argmax, stream);
    case 2: return launch_network_b<2>(x, n, d, th, kind, net, c, counts, argmax, stream);
    case 3: return launch_network_b<3>(x, n, d, th, kind, net, c, counts, argmax, stream);
    case 4: return launch_network_b<4>(x, n, d, th, kind, net, c, counts, argmax, stream);
    case 5: return launch_network_b<5>(x, n, d, th, kind, net, c, counts, argmax, stream);
    case 6: return launch_network_b<6>(x, n, d, th, kind, net, c, counts, argmax, stream);
    case 7: return launch_network_b<7>(x, n, d, th, kind, net, c, counts, argmax, stream);
    case 8: return launch_network_b<8>(x, n, d, th, kind, net, c, counts, argmax, stream);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_column_layer(const uint64_t *in, int32_t w_in, int32_t W, const int32_t *conn,
                               const uint64_t *tables, int32_t w_out, int32_t k, uint64_t *out,
                               const uint8_t *fanin, hipStream_t stream)
{
    switch (k) {
    case 1: return launch_layer_k<1>(in, w_in, conn, tables, w_out, out, W, fanin, stream);
    case 2: return launch_layer_k<2>(in, w_in, conn, tables, w_out, out, W, fanin, stream);
    case 3: return launch_layer_k<3>(in, w_in, conn, tables, w_out, out, W, fanin, stream);
    case 4: return launch_layer_k<4>(in, w_in, conn, tables, w_out, out, W, fanin, stream);
    case 5: return launch_layer_k<5>(in, w_in, conn, tables, w_out, out, W, fanin, stream);
    case 6: return launch_layer_k<6>(in, w_in, conn, tables, w_out, out, W, fanin, stream);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_column_head(const uint64_t *in, int32_t w_in, const int32_t *conn,
                              const uint64_t *tables, int32_t w_out, int32_t k, int32_t c,
                              int64_t n, const ColumnHeadPlan &hp, int32_t *counts,
                              int32_t *argmax, const uint8_t *fanin, hipStream_t stream)
{
    const int32_t g = w_out / c;
    auto run = [&](auto kc) {
        return launch_head_k<decltype(kc)::value>(in, w_in, conn, tables, g, c, n, hp, counts,
                                                  argmax, fanin, stream);
    };
    switch (k) {
    case 1: return run(std::integral_constant<int, 1>{});
    case 2: return run(std::integral_constant<int, 2>{});
    case 3: return run(std::integral_constant<int, 3>{});
    case 4: return run(std::integral_constant<int, 4>{});
    case 5: return run(std::integral_constant<int, 5>{});
    case 6: return run(std::integral_constant<int, 6>{});
    default: return hipErrorInvalidValue;
    }
}

}  // namespace bl
