// CRC registers on the matrix cores.
//
// A CRC register is linear over GF(2) in the bits of its message: bit m of it is the parity of the
// message bits that a fixed mask picks.  Parities come out of an ordinary matrix product: with
// bits as the numbers 0 and 1 (times powers of two) the product counts the ones a mask picks, exactly,
// and the count's lowest bit is the parity.  v_mfma_f32_32x32x64_f8f6f4 on 4-bit floats takes one dword of
// every lane -- lanes n and n + 32 are the two halves of the 64-long rows of column n -- against
// a 32 x 64 matrix of weights, one row for every bit of the register: 32 clocks of a SIMD's matrix
// core for the 256 bytes that four lookups a lane in byte tables took about 23 clocks of the whole
// compute unit's LDS for, whose 64 random addresses collide.  Its operands cost five vector
// instructions a dword, its weights one conflict-free 16-byte LDS read a lane.
//
// The code of a 4-bit float: 0001 is 0.5, 0010 1, 0100 2, 0110 4.  Bits 0, 1 and 2 of every nibble of a
// dword are such numbers where they stand, bit 3 after a shift by one; the weights 4, 2, 1 and 1 make
// every product of ones 2.  Sums stay below 2^24, and 2^24 + 2 * count holds the parity in its lowest bit.
#pragma once
#include "fold.h"

namespace ffsnap {

typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Words of the weights of one dword position: four for every lane.
constexpr int kWeightWords = 4 * 64;

// One dword of every lane.
__device__ __forceinline__ void matrix_add(f32x16& acc, const u32x4 weights, const uint32_t x)
{
    const i32x8 a = {int(weights.x), int(weights.y), int(weights.z), int(weights.w), 0, 0, 0, 0};
    const i32x8 b = {int(x & 0x11111111u), int(x & 0x22222222u), int(x & 0x44444444u),
                     int((x >> 1) & 0x44444444u), 0, 0, 0, 0};
    constexpr int kFloat4 = 4;
    acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, acc, kFloat4, kFloat4, 0, 0, 0, 0);
}

// Half a register per lane, in the upper 16 bits: lane n < 32 bits 16..31 of column n's, lane n + 32
// bits 0..15 of it, so times x^16.
__device__ __forceinline__ uint32_t matrix_halves(const f32x16& acc)
{
    uint32_t r = 0;
    static_for<16>([&](auto g) {
        r = __builtin_amdgcn_alignbit(__float_as_uint(acc[int(g)] + 16777216.0f), r, 1);
    });
    return r & 0xFFFF0000u;
}

// a * b where a has its upper 16 bits only.
__device__ __forceinline__ uint32_t gf2_mul_half(uint32_t a, uint32_t b)
{
    uint32_t p = 0;
#pragma unroll
    for (int i = 0; i < 16; i++) {
        p ^= (a & 0x80000000u) ? b : 0u;
        a <<= 1;
        b = gf2_mulx(b);
    }
    return p;
}

// The factor that lane `lane`'s half of its column's register still needs, where a column (lanes n
// and n + 32) is multiplied by x^(shift * (31 - n)).
inline uint32_t matrix_lane_factor(int lane, uint64_t shift)
{
    return gf2_xpow(shift * (31 - lane % 32) + (lane < 32 ? 0 : 16));
}

// Weights of one dword position (host; out: kWeightWords words): lanes below 32 hold dwords that
// enter the column's register times low, the others times high.
inline void build_matrix_weights(uint32_t* out, uint32_t low, uint32_t high)
{
    constexpr uint32_t kCode[4] = {6, 4, 2, 2};
    for (int half = 0; half < 2; half++) {
        uint32_t product[32];  // of bit b of a dword, x^(31 - b), and the factor
        uint32_t v = half ? high : low;
        for (int b = 31; b >= 0; b--, v = gf2_mulx(v)) product[b] = v;
        for (int m = 0; m < 32; m++) {
            // row m of the product comes out in lanes (m / 4) % 2 * 32 + n, at place g
            const int g = m / 8 * 4 + m % 4, bit = (m / 4) % 2 ? g : 16 + g;
            uint32_t* const w = out + 4 * (32 * half + m);
            w[0] = w[1] = w[2] = w[3] = 0;
            for (int b = 0; b < 32; b++)
                if ((product[b] >> bit) & 1u) w[b % 4] |= kCode[b % 4] << (4 * (b / 4));
        }
    }
}

}  // namespace ffsnap
