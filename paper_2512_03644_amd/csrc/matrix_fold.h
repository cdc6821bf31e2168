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
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Words of the weights of one dword position: four for every lane.
constexpr int kWeightWords = 4 * 64;

// A dword's bits as 4-bit floats, and weights as an operand.
__device__ __forceinline__ i32x8 matrix_bits(const uint32_t x)
{
    return i32x8{int(x & 0x11111111u), int(x & 0x22222222u), int(x & 0x44444444u),
                 int((x >> 1) & 0x44444444u), 0, 0, 0, 0};
}
__device__ __forceinline__ i32x8 matrix_weights(const u32x4 w)
{
    return i32x8{int(w.x), int(w.y), int(w.z), int(w.w), 0, 0, 0, 0};
}
constexpr int kFloat4 = 4;  // the operands' format

// One dword of every lane.
__device__ __forceinline__ void matrix_add(f32x16& acc, const u32x4 weights, const uint32_t x)
{
    acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(matrix_weights(weights), matrix_bits(x), acc, kFloat4,
                                                          kFloat4, 0, 0, 0, 0);
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

// The same with the multiples of b known beforehand: times[i] = b * x^i.
__device__ __forceinline__ void gf2_multiples(uint32_t (&times)[16], uint32_t b)
{
    static_for<16>([&](auto i) {
        times[i] = b;
        b = gf2_mulx(b);
    });
}
__device__ __forceinline__ uint32_t gf2_mul_half(const uint32_t a, const uint32_t (&times)[16])
{
    uint32_t p[2] = {0, 0};
    static_for<16>([&](auto i) { p[i % 2] ^= static_cast<uint32_t>(static_cast<int32_t>(a << i) >> 31) & times[i]; });
    return p[0] ^ p[1];
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

// ---- four streams at once ------------------------------------------------------------------------
//
// v_mfma_f32_16x16x128_f8f6f4: lanes n, n + 16, n + 32 and n + 48 are the quarters of column n, a product
// has 16 rows, so two of them make a register.  Twice the weights for a dword, but a product's sums
// take 4 registers a lane and not 16, so that several streams can use weights that have been read
// once; and a column's register comes out in four lanes, eight bits each, which suits four
// streams: the lanes share the streams out among themselves, and the multiplication by a lane's own
// factor, 130 instructions, is done once and not once per stream.

// Words of the weights of one dword position: two products, four words for every lane.
constexpr int kQuarterWords = 2 * 4 * 64;

struct QuarterSums {
    f32x4 p[2];  // the two products
};
__device__ __forceinline__ void matrix_add(QuarterSums& acc, const u32x4 (&weights)[2], const uint32_t x)
{
    const i32x8 b = matrix_bits(x);
    static_for<2>([&](auto s) {
        acc.p[s] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(matrix_weights(weights[s]), b, acc.p[s], kFloat4,
                                                                    kFloat4, 0, 0, 0, 0);
    });
}

// The eight bits of a stream's register that this lane has, from above into r.
__device__ __forceinline__ void matrix_take(uint32_t& r, const QuarterSums& acc)
{
    static_for<2>([&](auto s) {
        static_for<4>([&](auto g) {
            r = __builtin_amdgcn_alignbit(__float_as_uint(acc.p[s][int(g)] + 16777216.0f), r, 1);
        });
    });
}

// r: taken from streams 0 to 3, so byte j has bits 8 q .. 8 q + 7 of stream j's register, q = lane / 16.
// Lanes of row j (of 16) get what adds up over the row to the register of stream j, the columns
// times their factors: c0 of this lane for stream 0, c for the others.
__device__ __forceinline__ uint32_t matrix_streams(const uint32_t r, uint32_t c0, uint32_t c)
{
    uint32_t v[4] = {0, 0, 0, 0};
    static_for<8>([&](auto i) {
        static_for<4>([&](auto j) {
            const uint32_t on = static_cast<uint32_t>(static_cast<int32_t>(r << (24 - 8 * j + i)) >> 31);
            v[j] ^= on & (j == 0 ? c0 : c);
        });
        if constexpr (i < 7) { c0 = gf2_mulx(c0); c = gf2_mulx(c); }
    });
    const auto a = __builtin_amdgcn_permlane32_swap(v[0], v[2], false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(v[1], v[3], false, false);
    const auto w = __builtin_amdgcn_permlane16_swap(a[0] ^ a[1], b[0] ^ b[1], false, false);
    return w[0] ^ w[1];
}

// r: taken from streams 0 to 3, so byte j has bits 8 q .. 8 q + 7 of stream j's register, q = lane / 16.
// Lane 16 j + n gets the register of stream j's column n.
__device__ __forceinline__ uint32_t matrix_share(const uint32_t r, const int lane)
{
    // every lane gets r of all four quarters: the halves of a swapped pair of copies, twice
    const auto h = __builtin_amdgcn_permlane32_swap(r, r, false, false);
    const auto lo = __builtin_amdgcn_permlane16_swap(h[0], h[0], false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(h[1], h[1], false, false);
    // and takes byte j of each (0x0C: a byte of zeros)
    const uint32_t j = static_cast<uint32_t>(lane) >> 4, pick = j | (4 + j) << 8;
    return __builtin_amdgcn_perm(lo[1], lo[0], pick | 0x0C0C0000u) |
           __builtin_amdgcn_perm(hi[1], hi[0], pick << 16 | 0x0C0Cu);
}

// XOR over each 16 lanes, the same value in all of them.
__device__ __forceinline__ uint32_t row_xor(uint32_t v)
{
    v ^= __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true);   // quad_perm [1,0,3,2]: lane ^ 1
    v ^= __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true);   // quad_perm [2,3,0,1]: lane ^ 2
    v ^= __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, true);  // row_half_mirror: the other quad
    v ^= __builtin_amdgcn_mov_dpp(v, 0x140, 0xF, 0xF, true);  // row_mirror: the other eight
    return v;
}

// Weights of one dword position (host; out: kQuarterWords words): the dwords of the lanes of quarter q
// enter their column's register times factor * step^(3 - q).
inline void build_quarter_weights(uint32_t* out, uint32_t factor, uint32_t step)
{
    constexpr uint32_t kCode[4] = {6, 4, 2, 2};
    for (int quarter = 3; quarter >= 0; quarter--, factor = gf2_mul(factor, step)) {
        uint32_t product[32];
        uint32_t v = factor;
        for (int b = 31; b >= 0; b--, v = gf2_mulx(v)) product[b] = v;
        for (int s = 0; s < 2; s++)
            for (int m = 0; m < 16; m++) {
                // row m of product s comes out in the lanes of quarter m / 4, at place m % 4
                const int bit = 8 * (m / 4) + 4 * s + m % 4;
                uint32_t* const w = out + 4 * (64 * s + 16 * quarter + m);
                w[0] = w[1] = w[2] = w[3] = 0;
                for (int b = 0; b < 32; b++)
                    if ((product[b] >> bit) & 1u) w[b % 4] |= kCode[b % 4] << (4 * (b / 4));
            }
    }
}

}  // namespace ffsnap
