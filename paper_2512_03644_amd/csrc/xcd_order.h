// Order in which the workgroups of a launch take their tiles on a GPU with 8 XCDs.  No HIP
// dependency: the host tests include this file as well.
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#define FF_XCD_HD __host__ __device__
#else
#define FF_XCD_HD
#endif

namespace ffsnap {

// Workgroups are dealt to the 8 XCDs round-robin by launch index.  Within every complete round
// of 8 * g workgroups, workgroup b takes position (b mod 8) * g + b div 8 of the round, so the
// g workgroups that land on one XCD take g consecutive positions.  What is left behind the last
// complete round is divided the same way with runs of g / 2, then g / 4, ... so that a launch
// shorter than a round still gets the longest runs that fit.  A bijection on [0, n); the identity
// when g == 0.  g <= 2^28, so that 8 * g fits.
//
// Every wavefront computes this before its first load.  Runs are powers of two unless a caller names
// another length.  The rounds behind the complete ones of a power of two are then the bits of n below: the one of
// 8 * 2^l is there if that bit of n is set, and its workgroups are those whose number has the same bits above and a
// zero there.  So the highest bit in which b and n differ names b's round.  (Round by round by shifts, a short
// launch started half a microsecond later, by divisions a whole one.)
FF_XCD_HD inline uint32_t xcd_order(uint32_t b, uint32_t n, uint32_t g)
{
    constexpr uint32_t kXcds = 8, kXcdsLog2 = 3;
    if (!(g & (g - 1))) {
        const uint32_t bit = 31 - static_cast<uint32_t>(__builtin_clz(b ^ n));  // b < n
        if (g == 0 || bit < kXcdsLog2) return b;
        const uint32_t longest = 31 - static_cast<uint32_t>(__builtin_clz(g));
        const uint32_t l = bit - kXcdsLog2 < longest ? bit - kXcdsLog2 : longest;
        const uint32_t in = b & ((kXcds << l) - 1);
        return b - in + ((in & (kXcds - 1)) << l) + (in >> kXcdsLog2);
    }
    uint32_t start = 0;  // workgroups in front of the rounds of the current run length
    for (; g; g >>= 1) {
        const uint32_t span = kXcds * g;  // workgroups in one round over the XCDs
        const uint32_t full = (n - start) / span * span;
        if (b - start < full) {
            const uint32_t round = (b - start) / span, in = (b - start) % span;
            return start + round * span + (in % kXcds) * g + in / kXcds;
        }
        start += full;
    }
    return b;
}

#if defined(__HIPCC__)
// The same for the kernels, whose runs are all of a power of two, or none: without the code of other lengths.
__device__ inline uint32_t xcd_place(uint32_t b, uint32_t n, uint32_t g)
{
    __builtin_assume((g & (g - 1)) == 0);
    return xcd_order(b, n, g);
}
#endif

}  // namespace ffsnap
