// Thermometer encoder + bit-pack on gfx950.
//
// Wire f*b + t of sample s is (x[s][f] > theta[f][t]) (Sec. 3 "Encoders and
// heads"; App. A "Initialization"), packed 64 samples per 64-bit word along
// the batch (App. C.1 "Bit-packed inference").
//
// Two kernels, one lane per sample and one wave per 64-sample column in both:
//
// k_encode_t (b <= 8, the hot path).  A block owns a tile of features and
// packs one or two tiles of 16 columns (1024 samples) of them; each wave packs 4
// of the 16 columns, one at a time (at small batches 2 or 4 blocks share a
// tile's columns, down to one per wave, so that more blocks share the latency).
// A lane loads its own sample's feature bytes (16-byte loads where rows and
// tiles allow; the next column's bytes are in flight while the current one is
// packed) and compares them four at a time as bytes of a register
// (row_thermometer) into the 64-bit row of its sample's wires, and a 64x64 bit
// transpose across the wave (v_permlane32_swap for the 32-lane halves, then
// five ds_swizzle xor stages) turns rows of samples into packed words of wires:
// lane p ends with the word of wire row_wire(p).  The words of a 16-column tile
// are collected in LDS and written as whole 128-byte row segments.
//
// What bounds it: at large batches the pixel lines and the stores (1.51 GB at
// 2^18 x 3072, b = 7, in 367 us, 4.1 TB/s; torch copies at 4.8 on the same
// card), whatever the packing costs: with the codes looked up in an LDS table
// per block it took the same 367 us there, but 340 and 364 at b = 5 and 6
// against 307 and 339 now.  Small batches are latency, where the table's build
// and its lookups were a third: 16384 x 784 at b = 7 14.7 -> 9.1 us, 8192 x 3072
// at b = 3 16.5 -> 8.7, 65536 x 3072 at b = 3 59 -> 49.
//
// k_encode_ballot (any b <= 64).  Each comparison is a wave64 ballot, i.e. the
// packed word of one wire; v_writelane collects 64 such words into one lane
// each before they are stored.
//
// Both write either the row-major layout [wires][W] of bitlogic_encode or the
// slab layout [Wp/S][wires][S] of bitlogic_forward's intermediates.
//
// The binary-coded uniform fixed-point encoder (Sec. 3 "Encoders and heads":
// 2^b levels on b wires; Sec. 5 "Encoder") is the same kernel with another row
// (row_binary): round(v (2^b - 1) / 255), wire t = bit t.
#include <type_traits>

#include "bl_device.h"
#include "encode_row.h"

namespace bl {
namespace {

using namespace dev;

constexpr int kThreads = 256;

#ifndef BL_ENC_TPB
#define BL_ENC_TPB 2
#endif

template <int LAYOUT>
__device__ __forceinline__ int64_t out_index(int64_t wire, int64_t wb, int64_t W, int64_t rows)
{
    if constexpr (LAYOUT == kLayoutSlab)
        return slab_index(wire, wb, rows);
    else
        return wire * W + wb;
}

constexpr int kEncCols = 16;     // columns per output tile: 128-byte row segments
constexpr int kOtRow = kEncCols + 1;   // LDS words per tile row (odd: no bank conflicts)

// kDw dwords from a row of pixels.  vec16 (wave-uniform): 16-byte aligned.
template <int kDw>
__device__ __forceinline__ void load_row(const uint8_t *__restrict__ row, int vec16,
                                         uint32_t (&px)[kDw])
{
    if constexpr (kDw % 4 == 0) {
        if (vec16) {
#pragma unroll
            for (int q = 0; q < kDw / 4; ++q) {
                const u32x4 v = reinterpret_cast<const u32x4 *>(row)[q];
                px[4 * q + 0] = v.x;
                px[4 * q + 1] = v.y;
                px[4 * q + 2] = v.z;
                px[4 * q + 3] = v.w;
            }
            return;
        }
    }
#pragma unroll
    for (int q = 0; q < kDw; ++q)
        px[q] = load_u32(row + 4 * q);
}

// This lane's kDw pixel dwords (features f0 .. f0 + 4*kDw - 1 of sample s);
// zero past the batch or past the nf features of the tile.  full and inside
// are wave-uniform: the tile holds 4*kDw features; the column's 64 samples are
// all in the batch.
template <int kDw>
__device__ __forceinline__ void load_pixels(const uint8_t *__restrict__ x, int64_t s, int64_t n,
                                            int32_t d, int f0, int nf, int vec16, bool full,
                                            bool inside, uint32_t (&px)[kDw])
{
    if (full && inside) {
        load_row<kDw>(x + s * d + f0, vec16, px);
    } else if (full) {
        load_row<kDw>(x + min(s, n - 1) * d + f0, vec16, px);
#pragma unroll
        for (int q = 0; q < kDw; ++q)
            px[q] = s < n ? px[q] : 0u;
    } else {
        // rows shorter than a tile
        const uint8_t *row = x + s * d + f0;
#pragma unroll
        for (int q = 0; q < kDw; ++q) {
            uint32_t v = 0;
            if (s < n) {
                if (4 * q + 4 <= nf) {
                    v = load_u32(row + 4 * q);
                } else {
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (4 * q + u < nf)
                            v |= (uint32_t)row[4 * q + u] << (8 * u);
                }
            }
            px[q] = v;
        }
    }
}

template <int B, int LAYOUT, int KG, int CS>
__global__ __launch_bounds__(kThreads) void k_encode_t(
    const uint8_t *__restrict__ x, int64_t n, int32_t d, const uint8_t *__restrict__ th,
    uint64_t *__restrict__ out, int64_t W, int64_t W_cols, int32_t n_ftiles,
    int32_t tiles_per_block, int64_t n_tiles, int64_t n_tgroups, int vec16, int kind, int nt)
{
    using G = EncGeom<B, KG>;
    constexpr int kWires = G::kG * G::kWPG;              // wire rows of one output tile
    __shared__ __attribute__((aligned(16))) uint32_t s_nt[G::kG][16];
    __shared__ uint64_t otile[kWires * kOtRow];

    int tg, ft;
    if (!dealt_task(blockIdx.x, (int)n_tgroups, n_ftiles, tg, ft))
        return;
    // the last tile of rows that are no whole number of tiles starts earlier
    // and repeats `skip` features of the one before, which it does not write:
    // every tile's loads are then whole and rows need no alignment.  Loads
    // guarded per dword (per byte in rows that are not whole dwords) went out
    // one by one: 99991 x 3071 pixels at b = 3 took 1071 us against 207,
    // 50021 x 1021 at b = 6 185 against 42, 100000 x 3060 at b = 3 154
    // against 145; rows of whole 16-byte pieces and tiles are as they were
    const int f0 = max(min(ft * G::kFT, d - G::kFT), 0);
    const int skip = ft * G::kFT - f0;
    const int nf = min(G::kFT, d - f0);
    const int64_t D0 = (int64_t)d * B;
    const int lane = threadIdx.x % kWave;
    const int wave = threadIdx.x / kWave;

    // complements of the tile's thresholds, a dword per quad and wire (a
    // feature past the row gets 255, which nothing is above)
    if (kind == kEncThermometer) {
        for (int e = threadIdx.x; e < G::kG * G::kS; e += kThreads) {
            const int f = e / G::kS * G::kFPG + e % G::kS / B * 4, t = e % G::kS % B;
            uint32_t v = 0;
#pragma unroll
            for (int u = 0; u < 4; ++u)
                v |= (f + u < nf ? (uint32_t)th[(int64_t)(f0 + f + u) * B + t] : 255u) << (8 * u);
            s_nt[e / G::kS][e % G::kS] = ~v;
        }
        __syncthreads();
    }
    uint32_t mk[8];
    row_masks(mk);
    const dev::Transpose tr = transpose_consts(lane);
    const int my_wire = row_wire<B>(lane);

    // block tg covers part (tg % CS) of the columns of tile group tg / CS:
    // cpb columns per tile, cpw consecutive columns per wave
    constexpr int cpb = kEncCols / CS;
    constexpr int cpw = cpb / (kThreads / kWave);
    static_assert(cpw >= 1, "at least one column per wave");
    const int part = tg % CS;
    const int c_first = part * cpb + wave * cpw;      // this wave's first column of a tile
    const int64_t t0 = (int64_t)(tg / CS) * tiles_per_block;
    const int64_t t1 = min(t0 + tiles_per_block, n_tiles);
    const bool full = nf == G::kFT;
    auto inside = [&](int64_t gcol) { return (gcol + 1) * kWave <= n; };
    uint32_t px[G::kDw];
    {
        const int64_t gcol = t0 * kEncCols + c_first;
        load_pixels<G::kDw>(x, gcol * kWave + lane, n, d, f0, nf, vec16, full, inside(gcol),
                            px);
    }
    for (int64_t tile = t0; tile < t1; ++tile) {
        for (int cw = 0; cw < cpw; ++cw) {
            const int col = c_first + cw;                  // column inside the tile
            // prefetch the next column's pixels while this one is packed
            uint32_t nx[G::kDw];
            const bool more = cw + 1 < cpw || tile + 1 < t1;
            if (more) {
                const int64_t ncol = (cw + 1 < cpw) ? tile * kEncCols + col + 1
                                                    : (tile + 1) * kEncCols + c_first;
                load_pixels<G::kDw>(x, ncol * kWave + lane, n, d, f0, nf, vec16, full,
                                    inside(ncol), nx);
            }
#pragma unroll
            for (int gi = 0; gi < G::kG; ++gi) {
                uint32_t lo, hi;
                if (kind == kEncThermometer) {
                    // read here, not kept over the column loop: the registers
                    // that all groups' thresholds would take cost a wave per
                    // SIMD (397 against 367 us at 2^18 x 3072, b = 7)
                    asm volatile("" ::: "memory");
                    uint32_t nt[16];
#pragma unroll
                    for (int q = 0; q < (G::kS + 3) / 4; ++q) {
                        const u32x4 v = reinterpret_cast<const u32x4 *>(s_nt[gi])[q];
                        nt[4 * q] = v.x;
                        nt[4 * q + 1] = v.y;
                        nt[4 * q + 2] = v.z;
                        nt[4 * q + 3] = v.w;
                    }
                    row_thermometer<B>(px + gi * G::kQ, nt, mk, lo, hi);
                } else {
                    row_binary<B>(px + gi * G::kQ, mk, lo, hi);
                }
                transpose64(lo, hi, tr);
                if (my_wire >= 0)
                    otile[(gi * G::kWPG + my_wire) * kOtRow + col] = ((uint64_t)hi << 32) | lo;
            }
            if (more) {
#pragma unroll
                for (int q = 0; q < G::kDw; ++q)
                    px[q] = nx[q];
            }
        }
        __syncthreads();
        // write the tile: each wire's 16 words are one contiguous row segment
        const int64_t wb0 = tile * kEncCols;
        auto write = [&](auto stream) {
            for (int e = threadIdx.x; e < kWires * (cpb / 2); e += kThreads) {
                const int r = e / (cpb / 2);                   // tile wire row
                const int c2 = part * cpb + 2 * (e % (cpb / 2));   // even column
                const int gi = r / G::kWPG, p = r % G::kWPG;
                const int fg = gi * G::kFPG + p / B;           // feature of this wire in the tile
                const int64_t wb = wb0 + c2;
                if (fg < skip || fg >= nf || wb >= W_cols)
                    continue;
                const int64_t wire = (int64_t)(f0 + gi * G::kFPG) * B + p;
                const uint64_t w0 = otile[r * kOtRow + c2], w1 = otile[r * kOtRow + c2 + 1];
                uint64_t *q = out + out_index<LAYOUT>(wire, wb, W, D0);
                if (wb + 1 < W_cols && (LAYOUT == kLayoutSlab || ((uintptr_t)q % 16) == 0)) {
                    const u32x4 v = u32x4{(uint32_t)w0, (uint32_t)(w0 >> 32), (uint32_t)w1,
                                          (uint32_t)(w1 >> 32)};
                    if constexpr (decltype(stream)::value)
                        __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(q));
                    else
                        *reinterpret_cast<u32x4 *>(q) = v;
                } else {
                    q[0] = w0;
                    if (wb + 1 < W_cols)
                        out[out_index<LAYOUT>(wire, wb + 1, W, D0)] = w1;
                }
            }
        };
        if (nt)
            write(std::true_type{});
        else
            write(std::false_type{});
        __syncthreads();       // tile written before the next one reuses it
    }
}

constexpr int kBFeat = 32;             // features per tile
constexpr int kBRow = kBFeat + 4;      // LDS bytes per staged sample row (9 dwords)
constexpr int kBCols = 16;             // 64-sample columns per tile
constexpr int kBSamples = kBCols * kWave;

template <bool kAligned4, int LAYOUT>
__global__ __launch_bounds__(kThreads) void k_encode_ballot(
    const uint8_t *__restrict__ x, int64_t n, int32_t d,
    const uint8_t *__restrict__ th, int32_t b, uint64_t *__restrict__ out,
    int64_t W, int64_t W_cols, int32_t n_ftiles, int64_t n_cgroups)
{
    __shared__ uint8_t xs[kBSamples * kBRow];
    __shared__ uint8_t ths[kBFeat * 64];

    int cg, ft;
    if (!dealt_task(blockIdx.x, (int)n_cgroups, n_ftiles, cg, ft))
        return;
    const int f0 = ft * kBFeat;
    const int nf = min(kBFeat, d - f0);
    const int64_t s0 = (int64_t)cg * kBSamples;
    const int64_t D0 = (int64_t)d * b;

    for (int q = threadIdx.x; q < nf * b; q += kThreads)
        ths[q] = th[(int64_t)f0 * b + q];
    if (kAligned4) {
        for (int q = threadIdx.x; q < kBSamples * (kBFeat / 4); q += kThreads) {
            const int r = q / (kBFeat / 4), dw = q % (kBFeat / 4);
            const int64_t s = s0 + r;
            uint32_t v = 0;
            if (s < n && 4 * dw < nf)
                v = *reinterpret_cast<const uint32_t *>(x + s * d + f0 + 4 * dw);
            *reinterpret_cast<uint32_t *>(&xs[r * kBRow + 4 * dw]) = v;
        }
    } else {
        for (int q = threadIdx.x; q < kBSamples * kBFeat; q += kThreads) {
            const int r = q / kBFeat, f = q % kBFeat;
            const int64_t s = s0 + r;
            xs[r * kBRow + f] = (s < n && f < nf) ? x[s * d + f0 + f] : 0;
        }
    }
    __syncthreads();

    const int lane = threadIdx.x % kWave;
    const int wave = threadIdx.x / kWave;
    const int nwires = nf * b;
    const int64_t wire0 = (int64_t)f0 * b;
    for (int c = wave; c < kBCols; c += kThreads / kWave) {
        const int64_t col = (int64_t)cg * kBCols + c;
        if (col >= W_cols)
            break;
        const uint8_t *xrow = &xs[(c * kWave + lane) * kBRow];
        uint32_t acc_lo = 0, acc_hi = 0;
        int q = 0;
        for (int f = 0; f < nf; ++f) {
            const uint32_t xv = xrow[f];
            for (int t = 0; t < b; ++t, ++q) {
                const uint64_t m = __ballot(xv > (uint32_t)ths[f * b + t]);
                const int pos = q & (kWave - 1);
                acc_lo = (uint32_t)bl_writelane((int)(uint32_t)m, pos, (int)acc_lo);
                acc_hi = (uint32_t)bl_writelane((int)(uint32_t)(m >> 32), pos, (int)acc_hi);
                if (pos == kWave - 1) {
                    const int64_t wire = wire0 + (q - (kWave - 1)) + lane;
                    out[out_index<LAYOUT>(wire, col, W, D0)] = ((uint64_t)acc_hi << 32) | acc_lo;
                }
            }
        }
        const int rem = nwires & (kWave - 1);
        if (rem != 0 && lane < rem) {
            const int64_t wire = wire0 + (nwires - rem) + lane;
            out[out_index<LAYOUT>(wire, col, W, D0)] = ((uint64_t)acc_hi << 32) | acc_lo;
        }
    }
}

// Groups per tile: 32 to 64 features where the batch gives kEncBigBlocks blocks
// of them; half of that below (at b = 3 and b >= 5; one group at b <= 2 and two at
// b = 4 are not halved), for more blocks and a shorter chain in each (16384 x 784 at b = 7 13.7 -> 9.1 us; a quarter: 10.6; at 4096 blocks the big
// tiles win, 131072 x 784 at b = 7 43.8 against 46.4 us, and at 2^18 x 3072 368
// against 420, since more blocks share each pixel line).
constexpr int64_t kEncBigBlocks = 2048;
template <int B>
constexpr int big_groups()
{
    return B <= 2 ? 1 : B == 4 ? 2 : 4;
}
template <int B>
constexpr int small_groups()
{
    return big_groups<B>() < 2 ? 1 : 2;
}

template <int B, int LAYOUT, int KG, int CS>
hipError_t launch_tile(const uint8_t *x, int64_t n, int32_t d, const uint8_t *th, uint64_t *out,
                       int64_t W_cols, int kind, int64_t tpb, hipStream_t stream)
{
    using G = EncGeom<B, KG>;
    const int64_t W = (n + 63) / 64;
    const int64_t n_tiles = (W_cols + kEncCols - 1) / kEncCols;
    const int32_t n_ftiles = (d + G::kFT - 1) / G::kFT;
    const int64_t n_tg = (n_tiles + tpb - 1) / tpb * CS;
    const int64_t blocks = dealt_blocks(n_tg, n_ftiles);
    if (blocks > 0x7fffffff)
        return hipErrorInvalidConfiguration;
    const int vec16 = (d % 16 == 0) && ((uintptr_t)x % 16 == 0) && G::kFT % 16 == 0;
    hipLaunchKernelGGL((k_encode_t<B, LAYOUT, KG, CS>), dim3((unsigned)blocks), dim3(kThreads), 0,
                       stream, x, n, d, th, out, W, W_cols, n_ftiles, (int32_t)tpb, n_tiles, n_tg,
                       vec16, kind,
                       (int)streams_past_cache((int64_t)d * B * W_cols * 8));
    return hipGetLastError();
}

template <int B, int LAYOUT>
hipError_t launch_t(const uint8_t *x, int64_t n, int32_t d, const uint8_t *th, uint64_t *out,
                    int64_t W_cols, int kind, hipStream_t stream)
{
    constexpr int KB = big_groups<B>(), KS = small_groups<B>();
    const int64_t n_tiles = (W_cols + kEncCols - 1) / kEncCols;
    const int64_t big = n_tiles * ((d + EncGeom<B, KB>::kFT - 1) / EncGeom<B, KB>::kFT);
    // enough blocks to fill the chip; at most BL_ENC_TPB column tiles share one
    // block's constants (longer runs let the blocks that share pixel lines drift
    // apart, and the lines are fetched again: 2 tiles a block beat 1, 3, 4
    // and 8 on 256K-1M samples x 784-3072 features)
    if (big >= kEncBigBlocks) {
        int64_t tpb = big / kEncBigBlocks;
        tpb = tpb < 1 ? 1 : (tpb > BL_ENC_TPB ? BL_ENC_TPB : tpb);
        return launch_tile<B, LAYOUT, KB, 1>(x, n, d, th, out, W_cols, kind, tpb, stream);
    }
    // small batches: tiles of fewer features, and each tile's 16 columns split
    // over 2 or 4 blocks (down to one column per wave), so that more blocks
    // share the latency
    const int64_t small = n_tiles * ((d + EncGeom<B, KS>::kFT - 1) / EncGeom<B, KS>::kFT);
    if (2 * small < 1024)
        return launch_tile<B, LAYOUT, KS, 4>(x, n, d, th, out, W_cols, kind, 1, stream);
    if (small < 1024)
        return launch_tile<B, LAYOUT, KS, 2>(x, n, d, th, out, W_cols, kind, 1, stream);
    return launch_tile<B, LAYOUT, KS, 1>(x, n, d, th, out, W_cols, kind, 1, stream);
}

template <int LAYOUT>
hipError_t launch_ballot(const uint8_t *x, int64_t n, int32_t d, const uint8_t *th, int32_t b,
                         uint64_t *out, int64_t W_cols, hipStream_t stream)
{
    const int64_t W = (n + 63) / 64;
    const int32_t n_ftiles = (d + kBFeat - 1) / kBFeat;
    const int64_t n_cg = (W_cols + kBCols - 1) / kBCols;
    const int64_t blocks = dealt_blocks(n_cg, n_ftiles);
    if (blocks > 0x7fffffff)
        return hipErrorInvalidConfiguration;
    const bool aligned4 = (d % 4 == 0) && ((uintptr_t)x % 4 == 0);
    if (aligned4)
        hipLaunchKernelGGL((k_encode_ballot<true, LAYOUT>), dim3((unsigned)blocks), dim3(kThreads),
                           0, stream, x, n, d, th, b, out, W, W_cols, n_ftiles, n_cg);
    else
        hipLaunchKernelGGL((k_encode_ballot<false, LAYOUT>), dim3((unsigned)blocks),
                           dim3(kThreads), 0, stream, x, n, d, th, b, out, W, W_cols, n_ftiles,
                           n_cg);
    return hipGetLastError();
}

template <int LAYOUT>
hipError_t launch_layout(const uint8_t *x, int64_t n, int32_t d, const uint8_t *th, int32_t b,
                         uint64_t *out, int64_t W_cols, int kind, hipStream_t stream)
{
    switch (b) {
    case 1: return launch_t<1, LAYOUT>(x, n, d, th, out, W_cols, kind, stream);
    case 2: return launch_t<2, LAYOUT>(x, n, d, th, out, W_cols, kind, stream);
    case 3: return launch_t<3, LAYOUT>(x, n, d, th, out, W_cols, kind, stream);
    case 4: return launch_t<4, LAYOUT>(x, n, d, th, out, W_cols, kind, stream);
    case 5: return launch_t<5, LAYOUT>(x, n, d, th, out, W_cols, kind, stream);
    case 6: return launch_t<6, LAYOUT>(x, n, d, th, out, W_cols, kind, stream);
    case 7: return launch_t<7, LAYOUT>(x, n, d, th, out, W_cols, kind, stream);
    case 8: return launch_t<8, LAYOUT>(x, n, d, th, out, W_cols, kind, stream);
    default:
        if (kind != kEncThermometer)
            return hipErrorInvalidValue;          // binary codes have at most 8 bits
        return launch_ballot<LAYOUT>(x, n, d, th, b, out, W_cols, stream);
    }
}

}  // namespace

hipError_t launch_encode(const uint8_t *x, int64_t n, int32_t d, const uint8_t *thresholds,
                         int32_t b, uint64_t *out, int layout, int64_t W_cols,
                         hipStream_t stream, int kind)
{
    if (layout == kLayoutSlab)
        return launch_layout<kLayoutSlab>(x, n, d, thresholds, b, out, W_cols, kind, stream);
    return launch_layout<kLayoutRowMajor>(x, n, d, thresholds, b, out, W_cols, kind, stream);
}

}  // namespace bl
