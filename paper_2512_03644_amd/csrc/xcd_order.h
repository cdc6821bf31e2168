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
// another length, and go by shifts: with two divisions a round a short launch, which halves its run
// six or seven times, started 0.4-0.7 us later (verify of 3.2 MB 9.6 -> 8.9 us, pack of 32 MB 19.1 -> 18.7).
FF_XCD_HD inline uint32_t xcd_order(uint32_t b, uint32_t n, uint32_t g)
{
    constexpr uint32_t kXcds = 8, kXcdsLog2 = 3;
    uint32_t start = 0;  // workgroups in front of the rounds of the current run length
    if (g && !(g & (g - 1))) {
        for (int l = 31 - __builtin_clz(g); l >= 0; l--) {
            const uint32_t span_log2 = static_cast<uint32_t>(l) + kXcdsLog2;
            const uint32_t full = (n - start) >> span_log2 << span_log2;
            if (b - start < full) {
                const uint32_t in = (b - start) & ((1u << span_log2) - 1);
                return b - in + ((in & (kXcds - 1)) << l) + (in >> kXcdsLog2);
            }
            start += full;
        }
        return b;
    }
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

}  // namespace ffsnap
