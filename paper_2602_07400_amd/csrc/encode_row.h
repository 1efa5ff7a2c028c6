// The wire bits of one sample's features as 64-bit rows, shared by the encoders
// (Sec. 3 "Encoders and heads"; App. C.1 "Bit-packed inference").
#pragma once

#include "bl_device.h"

namespace bl {
namespace dev {

// A dword at any address (gfx950 global loads need no alignment).
__device__ __forceinline__ uint32_t load_u32(const uint8_t *p)
{
    uint32_t v;
    __builtin_memcpy(&v, p, sizeof v);
    return v;
}

// Features per 64-wire group of b wires each, in quads whose four bytes are
// compared at once: as many as fit, but one fewer at b = 3, so that a tile is a
// whole number of 16-byte pieces and shares 128-byte pixel lines with its
// neighbours instead of straddling them.
constexpr int group_quads(int b) { return b == 3 ? 4 : 16 / b; }

template <int B, int KG>
struct EncGeom {
    static constexpr int kQ = group_quads(B);            // quads per group
    static constexpr int kFPG = 4 * kQ;                  // features per group
    static constexpr int kS = kQ * B;                    // (quad, wire) slots per group
    static_assert(kS <= 16, "a group's wires fit one 64-bit row");
    static constexpr int kWPG = kFPG * B;                // wires per group (<= 64)
    static constexpr int kG = KG;                        // groups per tile
    static constexpr int kFT = kFPG * kG;                // features per tile
    static constexpr int kDw = kFT / 4;                  // pixel dwords per sample
};

// The wire bits of a group of features of one sample, as a 64-bit row: slot
// k = quad * B + t puts bit t of the quad's four features at bits 7 - k % 8,
// 15 - k % 8, ... of half k / 8.  Thermometer: byte x is above byte th exactly
// where x + ~th carries out of the byte, the majority of x, ~th and the sum of
// their low 7 bits at bit 7; four comparisons in three instructions (and, add,
// v_bitop3), two more to place them, all of the full-rate kind.  Binary code:
// round(v (2^B - 1) / 255) = (t + (t >> 8)) >> 8 with t = v (2^B - 1) + 128,
// two features per register.
template <int B>
__device__ __forceinline__ void place_slot(int k, uint32_t r, const uint32_t (&mk)[8],
                                           uint32_t &lo, uint32_t &hi)
{
    uint32_t &row = k < 8 ? lo : hi;
    // row | (r & mk): v_bitop3 with the mask in a VGPR
    row = __builtin_amdgcn_bitop3_b32(row, r, mk[k % 8], 0xF8);
}

template <int B>
__device__ __forceinline__ void row_thermometer(const uint32_t *px, const uint32_t (&nt)[16],
                                                const uint32_t (&mk)[8], uint32_t &lo,
                                                uint32_t &hi)
{
    using G = EncGeom<B, 1>;
    lo = hi = 0;
#pragma unroll
    for (int k = 0; k < G::kS; ++k) {
        const uint32_t v = px[k / B];
        const uint32_t z = (v & 0x7F7F7F7Fu) + (nt[k] & 0x7F7F7F7Fu);
        place_slot<B>(k, __builtin_amdgcn_bitop3_b32(v, nt[k], z, 0xE8) >> (k % 8), mk, lo, hi);
    }
}

template <int B>
__device__ __forceinline__ void row_binary(const uint32_t *px, const uint32_t (&mk)[8],
                                           uint32_t &lo, uint32_t &hi)
{
    using G = EncGeom<B, 1>;
    lo = hi = 0;
#pragma unroll
    for (int q = 0; q < G::kQ; ++q) {
        auto code = [](uint32_t v) {             // bytes 0 and 2 of v
            const uint32_t t = (v << B) - v + 0x00800080u;
            return ((t + ((t >> 8) & 0x00FF00FFu)) >> 8) & 0x00FF00FFu;
        };
        const uint32_t c = code(px[q] & 0x00FF00FFu) | code((px[q] >> 8) & 0x00FF00FFu) << 8;
#pragma unroll
        for (int t = 0; t < B; ++t) {
            const int k = q * B + t;
            // bit t of each byte to bit 7 - k % 8
            place_slot<B>(k, __builtin_amdgcn_alignbit(c, c, (t - 7 + k % 8 + 32) % 32), mk, lo,
                          hi);
        }
    }
}

// The wire (within its group) whose column lane p holds after the transpose, or
// -1 for an idle row bit.
template <int B>
__device__ __forceinline__ int row_wire(int p)
{
    const int slot = p / 32 * 8 + 7 - p % 8;
    return slot < EncGeom<B, 1>::kS ? (slot / B * 4 + p % 32 / 8) * B + slot % B : -1;
}

// row_*'s placement masks, kept in VGPRs: v_bitop3 runs at full rate on them
// (55 T lane-ops/s; 37 with an SGPR operand).
__device__ __forceinline__ void row_masks(uint32_t (&mk)[8])
{
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        mk[k] = 0x80808080u >> k;
        asm volatile("" : "+v"(mk[k]));
    }
}

}  // namespace dev
}  // namespace bl
