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
};

// Enqueues prepare (crcs = affine, zero tail, counter = 0) and the tile kernels.
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
