// Launch wrapper of the fused optimizer-step + snapshot kernels (fused.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.hpp"
#include "layout.hpp"

namespace ffsnap {

// Scalars shared by every element, derived on the host in double and rounded once to fp32.
struct AdamConsts {
    float decay, b1, omb1, b2, omb2, step_size, bc2s, eps;
};

struct FusedConsts {
    AdamConsts adam;
    float inv_scale = 1.0f;            // fp16 variant: reciprocal of the loss scale
    uint64_t* n_nonfinite = nullptr;   // fp16 variant: device counter of inf/NaN gradients, or null
    uint32_t xcd_group = 0;            // XCD-aware order of the work tiles (see xcd_order.h)
    // Chained step: master, m and v are read from this snapshot buffer (at the segments' stream
    // offsets) instead of their tensors, and those tensors are not written.  Null: in-place step.
    const uint8_t* prev = nullptr;
    uint32_t image = 0;  // in-place step: whole workgroups store their fp32 streams through LDS
    // A step in one launch (tally set): its contributions to crcs[] meet in words of the plan's, which are zero before
    // and after; workgroups from n_groups on clear the buffer's end and *n_nonfinite (open_count in tally.h).
    uint64_t* tally = nullptr;
    const StepTicket* runs = nullptr;
    const StepTicket* heads = nullptr;
    uint64_t* state = nullptr;
    uint64_t epoch = 0, payload = 0, buffer_bytes = 0;
    uint32_t affine = 0, n_groups = 0;
};

// Device table of the fused kernels (kFusedTabWords entries): weights (matrix_fold.h) of the dwords of two
// rows of 16-byte slots and of two rows of 8-byte slots, then lane constants: for k = 0..15 and every lane of a
// parameter sub-block, x^(8 * bytes between the end of the lane's column in its stream and the end of a
// row, plus k sub-blocks), and for k = 0..3 the same for the columns of a RAW sub-block's pairs of rows.
constexpr int kFusedWeightWords = 12 * 2 * 4 * 64;
constexpr int kFusedTabWords = kFusedWeightWords + 32 * 64 + 4 * 64;
void build_fused_tabs(uint32_t* tab);

// Gradient pointers of up to kGradsPerLaunch consecutive parameter groups, handed to the kernel by
// value in its arguments (16 KiB).  A step over more takes several launches, each with a ramp and a tail of its own
// and its share of the host's time: with 384 to a launch / with 2048, us, 2000 ragged groups of 115 million elements in fp16
// 1032 / 972, 27 million 292 / 235 (chained 224 / 171), 0.2 million 127 / 114, 500 groups of 6 million 70 / 63 (57 / 48).
constexpr uint32_t kGradsPerLaunch = 2048;
// Steps of up to so many workgroups go in one launch on the default stream, without the kernel that sets crcs[] and
// clears the buffer's end (2 us).  With it / without, us, in place: 10 workgroups 11.3 / 9.5, 128 12.3 / 10.1, 35 fp16
// parameters and 300 RAW tensors 24.6 / 23.5, 750 32.0 / 30.0, 1480 57.7 / 56.1, 2450 82.6 / 81.5, 2940 96.9 / 97.3;
// chained 750 30.4 / 24.6, 1480 44.4 / 40.2, 2450 62.6 / 59.3, 2940 73.1 / 72.6.  In longer launches a workgroup's
// returning atomics hold up the next one's start.
constexpr uint64_t kTallyStepGroups = 2560;
// Steps over buffers up to here load through the caches: what they read was written not long ago, and is still in the
// 256 MiB last-level cache, or would be by the next step.  Non-temporal / plain loads, us, one set of tensors and snapshots (as in a
// training program) and three in turn, in place 30 / 45 / 60 / 80 / 100 MB 24.4 / 33.6 / 44.1 / 55.2 / 66.4 against 21.0 / 31.8 /
// 39.2 / 48.4 / 57.6, in turn 24.4 / 33.8 / 44.4 / 55.4 / 66.7 against 21.3 / 32.3 / 39.5 / 53.1 / 71.5; chained 30 / 60 / 80 / 100 MB
// 22.1 / 32.3 / 41.4 / 49.5 against 17.5 / 27.7 / 34.1 / 41.1, in turn 22.6 / 33.3 / 42.4 / 50.8 against 18.6 / 27.6 / 38.6 /
// 51.9.  (The gradients alone non-temporal: 2-7 % behind either.)  RAW tensors as well, us: 0.2 million elements and 32 MB of them
// 19.6 / 18.9, chained 19.7 / 17.9, 2.1 million and 9 / 32 MB 22.8 / 36.9 against 21.5 / 32.0, chained 20.7 / 31.9 against 18.7 / 26.7;
// first passes over a new state 50.9 / 52.0 / 65.0 against 46.4 / 51.1 / 63.8, chained 47.4 / 52.0 / 56.8 against 44.6 / 52.8 / 54.3.
constexpr uint64_t kWarmStepBytes = 80ull << 20;
template <uint32_t N>
struct GradPtrsOf {
    uint64_t p[N];
};
using GradPtrs = GradPtrsOf<kGradsPerLaunch>;

// A plan's work lists on the device, and on the host where the part of every launch begins (one
// entry more than there are launches).
struct FusedWork {
    const WorkTile* tiles = nullptr;       // parameter tiles first, sorted by group, then RAW tiles
    const WorkWave* waves = nullptr;
    std::vector<uint32_t> launch_tile;     // parameter tiles only
    std::vector<uint32_t> launch_wave;
    std::vector<uint8_t> launch_off_lines; // most elements have an fp32 stream off the 128-byte lines
    // of a plan whose step may go in one launch
    const StepTicket* runs = nullptr;
    const StepTicket* heads = nullptr;
    uint64_t* tally = nullptr;
};

// Enqueues prepare (crcs = affine, zero tail, counter = 0) and the tile kernels; with consts.tally the tile kernel
// alone.
// tabs: device table (build_fused_tabs).  grads: HOST array of n_params device pointers, read
// during the call only.  f16: gradients and working weights are fp16 (else bf16).  bare: the
// step's traffic alone -- every parameter tile's loads and stores with no arithmetic and no CRC
// (16-bit weights := gradient bits, master, m, v unchanged); crcs, the RAW segments and the zero
// tail are not touched.
hipError_t launch_fused(bool f16, const FusedWork& work, const void* const* grads, uint32_t n_params,
                        const uint32_t* tabs, void* chunks, uint32_t* crcs, uint64_t n_chunks,
                        uint64_t payload, uint64_t buffer_bytes, uint32_t affine,
                        const FusedConsts& consts, bool bare, hipStream_t stream);

}  // namespace ffsnap
