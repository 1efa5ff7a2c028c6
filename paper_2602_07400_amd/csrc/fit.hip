// Quantile thermometer thresholds fitted on the device (Sec. 4
// "Initialization": fitted once from the empirical pixel quantiles of the
// training split; App. B: over the flattened pixel distribution).
//
// The d features are cut into n_groups contiguous groups (one group: the
// whole flattened distribution; one per colour channel for CHW images).  Per
// group, with cum(v) = number of the group's pixels <= v and total = n * d /
// n_groups, threshold i (i = 1..b) is the smallest v with
// (b + 1) * cum(v) >= i * total -- the exact integer form of
// cum(v) / total >= i / (b + 1) -- and every feature of the group receives
// the group's ladder.
//
// k_fit_hist: each block counts a run of rows into an LDS histogram per group
// (LDS atomics), then adds it into the global 64-bit histogram.  The LDS
// histogram holds R interleaved copies of every bin (lane l counts into copy l
// mod R, at word bin * R + l mod R); at R = 32, which up to 4 groups get, the 32
// lanes of half a wave fall into 32 banks, whatever the pixels.  The copies are
// summed before the global add.  A thread keeps a 16-byte column of the rows,
// with its bytes' groups, and walks the rows of its place in the block,
// kRowUnroll rows' loads at a time, at any alignment; the last column of rows
// that are no whole number of them starts earlier and counts only its own
// bytes.  k_fit_select: one block per group turns the histogram into the ladder
// (a block prefix sum, one thread per bin).
//
// What bounds it: the LDS atomics (about 11 lanes a clock and CU) at large
// batches, 805 MB in three groups in 148 us with all three launches (163 with
// 16 copies, dword columns and 1024 blocks of 256 threads), the global adds of
// the histograms at small ones: one round of 1024-thread blocks instead of 1024
// blocks took 25 MB from 38 to 21 us and 0.25 MB from 30 to 12; rows that are not
// whole dwords no longer go a byte per load (100000 x 2001 74 -> 43 us).  Two rows
// in flight a thread were as fast as 4 and 3-7% faster than 8.
#include "bl_internal.h"

namespace bl {
namespace {

constexpr int kThreads = 256;
constexpr int kHistThreads = 1024;
constexpr int kRowUnroll = 2;
constexpr int kFitMaxRep = 32;                    // copies of each histogram bin
constexpr int kFitHistBytes = 128 << 10;          // LDS of one histogram block
constexpr int kColBytes = 16;                     // pixels of a thread's column

__global__ __launch_bounds__(kThreads) void k_fit_clear(uint64_t *__restrict__ ws, int32_t n)
{
    const int i = blockIdx.x * kThreads + threadIdx.x;
    if (i < n)
        ws[i] = 0;
}

__global__ __launch_bounds__(kHistThreads) void k_fit_hist(
    const uint8_t *__restrict__ x, int64_t n, int32_t d, int32_t per, int32_t n_groups,
    int64_t rows_per_block, int32_t rep_log2, uint64_t *__restrict__ ws)
{
    extern __shared__ uint32_t hist[];             // [n_groups][256][R], R = 2^rep_log2
    const int nbins = n_groups * 256;
    for (int i = threadIdx.x; i < nbins << rep_log2; i += kHistThreads)
        hist[i] = 0;
    __syncthreads();
    const uint32_t copy = threadIdx.x & ((1u << rep_log2) - 1);
    const int64_t r0 = (int64_t)blockIdx.x * rows_per_block;
    const int64_t r1 = min(n, r0 + rows_per_block);
    if (d >= kColBytes) {
        // columns of 16 bytes; up to kHistThreads of them side by side, as many
        // rows at once as fit beside
        const int n_cols = (d + kColBytes - 1) / kColBytes;
        const int wide = min(n_cols, kHistThreads);
        const int tall = kHistThreads / wide;
        const int rt = threadIdx.x / wide;
        for (int c0 = 0; c0 < n_cols; c0 += wide) {
            const int c = c0 + threadIdx.x - rt * wide;
            if (rt >= tall || c >= n_cols)
                continue;
            const int off = min(c * kColBytes, d - kColBytes);
            const int first = c * kColBytes - off;       // bytes the column before counts
            uint32_t base[kColBytes];                    // word of bin 0 of each byte's group
#pragma unroll
            for (int u = 0; u < kColBytes; ++u)
                base[u] = ((uint32_t)((off + u) / per * 256) << rep_log2) + copy;
            // the bytes before `first` count as zeros, taken back below
            u32x4 own;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int drop = min(max(first - 4 * q, 0), 4);
                own[q] = drop == 4 ? 0u : ~0u << (8 * drop);
            }
            auto count = [&](u32x4 v) {
                v &= own;
#pragma unroll
                for (int u = 0; u < kColBytes; ++u)
                    atomicAdd(&hist[base[u] + (((v[u / 4] >> (8 * (u % 4))) & 0xFFu) << rep_log2)],
                              1u);
            };
            const uint8_t *src = x + off;
            int64_t r = r0 + rt;
            for (; r + (kRowUnroll - 1) * tall < r1; r += kRowUnroll * tall) {
                u32x4 v[kRowUnroll];
#pragma unroll
                for (int q = 0; q < kRowUnroll; ++q)
                    __builtin_memcpy(&v[q], src + (r + q * tall) * d, sizeof v[q]);
#pragma unroll
                for (int q = 0; q < kRowUnroll; ++q)
                    count(v[q]);
            }
            for (; r < r1; r += tall) {
                u32x4 v;
                __builtin_memcpy(&v, src + r * d, sizeof v);
                count(v);
            }
            if (first > 0 && r0 + rt < r1) {
                const uint32_t rows = (uint32_t)((r1 - r0 - rt + tall - 1) / tall);
#pragma unroll
                for (int u = 0; u < kColBytes; ++u)
                    if (u < first)
                        atomicSub(&hist[base[u]], rows);
            }
        }
    } else {
        for (int64_t e = threadIdx.x; e < (r1 - r0) * d; e += kHistThreads)
            atomicAdd(&hist[((uint32_t)((int)(e % d) / per * 256 + x[r0 * d + e]) << rep_log2) +
                            copy],
                      1u);
    }
    __syncthreads();
    // sum the copies (each thread starts at another copy, so that the
    // threads of a wave read different banks), then one global add per bin
    const int nrep = 1 << rep_log2;
    for (int i = threadIdx.x; i < nbins; i += kHistThreads) {
        uint32_t sum = 0;
        for (int k = 0; k < nrep; ++k)
            sum += hist[((uint32_t)i << rep_log2) + ((uint32_t)(k + i) & (uint32_t)(nrep - 1))];
        if (sum)
            atomicAdd(reinterpret_cast<unsigned long long *>(&ws[i]), (unsigned long long)sum);
    }
}

__global__ __launch_bounds__(kThreads) void k_fit_select(
    const uint64_t *__restrict__ ws, int64_t total, int32_t per, int32_t b,
    uint8_t *__restrict__ th)
{
    static_assert(kThreads == 256, "one thread per histogram bin");
    __shared__ uint64_t cum[256];
    __shared__ uint8_t ladder[64];
    const int grp = blockIdx.x;
    const int v = threadIdx.x;
    // inclusive prefix sum of the 256 bins (Hillis-Steele, 8 steps)
    cum[v] = ws[grp * 256 + v];
    __syncthreads();
#pragma unroll
    for (int off = 1; off < 256; off <<= 1) {
        const uint64_t add = v >= off ? cum[v - off] : 0;
        __syncthreads();
        cum[v] += add;
        __syncthreads();
    }
    // threshold i is the smallest v with (b + 1) cum(v) >= i total (255 if
    // none): thread v sets it where the criterion first holds
    const uint64_t b1 = (uint64_t)(b + 1);
    for (int i = 1; i <= b; ++i) {
        const uint64_t need = (uint64_t)i * (uint64_t)total;
        const bool here = cum[v] * b1 >= need;
        const bool before = v > 0 && cum[v - 1] * b1 >= need;
        if ((here && !before) || (v == 255 && !here))
            ladder[i - 1] = (uint8_t)v;
    }
    __syncthreads();
    uint8_t *dst = th + (int64_t)grp * per * b;
    for (int64_t e = threadIdx.x; e < (int64_t)per * b; e += kThreads)
        dst[e] = ladder[e % b];
}

}  // namespace

hipError_t launch_fit_quantiles(const uint8_t *x, int64_t n, int32_t d, int32_t b,
                                int32_t n_groups, uint8_t *th, uint64_t *ws, hipStream_t stream)
{
    if (n_groups < 1 || n_groups > kFitMaxGroups || d % n_groups != 0 || b < 1 || b > 64 ||
        n < 1)
        return hipErrorInvalidValue;
    const int32_t per = d / n_groups;
    const int32_t bins = n_groups * 256;
    hipLaunchKernelGGL(k_fit_clear, dim3((bins + kThreads - 1) / kThreads), dim3(kThreads), 0,
                       stream, ws, bins);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    // as many bin copies as the block's LDS budget allows (at least one)
    int32_t rep_log2 = 0;
    while ((2 << rep_log2) <= kFitMaxRep &&
           (size_t)bins * sizeof(uint32_t) * (2u << rep_log2) <= (size_t)kFitHistBytes)
        ++rep_log2;
    const size_t lds = ((size_t)bins << rep_log2) * sizeof(uint32_t);
    // one round of blocks: two a CU where their LDS allows, each of at least the
    // rows that its threads walk side by side (fewer leave threads idle and add
    // more histograms into memory: 784 features at 200 and 500 rows 15.0 and 21.3
    // us with one row a block, 12.7 so), and a block's count of any one bin (at
    // most rows * per) stays below 2^31
    const int64_t want = 256 * (2 * lds <= (160 << 10) ? 2 : 1);
    const int64_t n_cols = ((int64_t)d + kColBytes - 1) / kColBytes;
    const int64_t tall = n_cols < kHistThreads ? kHistThreads / n_cols : 1;
    int64_t rows = (n + want - 1) / want;
    if (rows < tall)
        rows = tall;
    const int64_t cap = ((int64_t)1 << 31) / per;
    if (rows > cap)
        rows = cap < 1 ? 1 : cap;
    const int64_t blocks = (n + rows - 1) / rows;
    if (blocks > 0x7fffffff)
        return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(k_fit_hist, dim3((unsigned)blocks), dim3(kHistThreads), lds, stream, x, n,
                       d, per, n_groups, rows, rep_log2, ws);
    e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(k_fit_select, dim3((unsigned)n_groups), dim3(kThreads), 0, stream, ws,
                       n * (int64_t)per, per, b, th);
    return hipGetLastError();
}

}  // namespace bl
