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
// when g == 0.  g is a power of two up to 2^28, so that 8 * g fits, or 0.
//
// Every wavefront computes this before its first load.  The rounds behind the complete ones are the bits of n below: the one of
// 8 * 2^l is there if that bit of n is set, and its workgroups are those whose number has the same bits above and a
// zero there.  So the highest bit in which b and n differ names b's round.  (Round by round by shifts, a short
// launch started half a microsecond later, by divisions a whole one.)
FF_XCD_HD inline uint32_t xcd_order(uint32_t b, uint32_t n, uint32_t g)
{
    constexpr uint32_t kXcds = 8, kXcdsLog2 = 3;
    const uint32_t bit = 31 - static_cast<uint32_t>(__builtin_clz(b ^ n));  // b < n
    if (g == 0 || bit < kXcdsLog2) return b;
    const uint32_t longest = 31 - static_cast<uint32_t>(__builtin_clz(g));
    const uint32_t l = bit - kXcdsLog2 < longest ? bit - kXcdsLog2 : longest;
    const uint32_t in = b & ((kXcds << l) - 1);
    return b - in + ((in & (kXcds - 1)) << l) + (in >> kXcdsLog2);
}

}  // namespace ffsnap
