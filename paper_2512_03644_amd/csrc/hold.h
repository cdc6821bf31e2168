// A restore that leaves damaged chunks out, in one pass over the buffer.
//
// A chunk may be scattered only when all of it has been checked, so the plain way reads the buffer twice:
// once to verify, once to scatter.  Here every wavefront keeps its 32 KiB tile in registers (128 of
// them), hands the tile's CRC register to its chunk's tally, waits for the chunk's verdict and scatters what it
// holds.  The chip holds 96 MB that way (three workgroups on a compute unit), 24 chunks of 4 MiB; at 3 TB/s read
// that is a lifetime of 30 us for a workgroup, of which the wait is a few.  3.2 GB of 20,000 ragged tensors 1560 ->
// 1179 us (a restore of all of it takes 1105; two workgroups on a compute unit 1269); other sizes at launch_hold().
//
// A chunk's workgroups are dealt to the XCDs in short runs, so that they start at about the same time; but
// nothing promises that all of them are in flight together (other kernels may hold compute units).  So a wait
// is bounded, and a wavefront whose patience ends reads the chunk and finds the verdict by itself, unless it comes
// meanwhile (find_verdict).
#pragma once
#include "fold.h"
#include "kernels.hpp"
#include "matrix_fold.h"
#include "tally.h"

namespace ffsnap {

namespace hold {

constexpr int kRows = 32;          // of a tile
constexpr int kBlocks = 4;         // of 8 rows, the unit of the weights
constexpr int kBlockRows = kRows / kBlocks;
constexpr int kWaves = 4;
constexpr int kThreads = kWaves * kWaveSize;
constexpr uint32_t kRowBytes = 1024, kTileBytes = kRows * kRowBytes;
constexpr int kRingWords = 520;    // two rows and 16 bytes, padded to a multiple of 16 bytes

struct HoldLds {
    u32x4 weight[kBlockRows * 4][kWaveSize];
    uint32_t ring[kWaves][kRingWords];
    uint64_t sum[kWaves];                   // per run, at its first wavefront's place (run_complete)
    uint32_t verdict[kWaves];               // ... 0: none yet, 2: sound, 3: damaged
};

// One 8 KiB block's sums.
template <class Row>
__device__ __forceinline__ f32x16 block_sums(const HoldLds& lds, const int lane, Row&& row)
{
    f32x16 acc = {};
    static_for<kBlockRows>([&](auto r) {
        const u32x4 w = row(r);
        static_for<4>([&](auto f) { matrix_add(acc, lds.weight[4 * r + f][lane], w[int(f)]); });
        __builtin_amdgcn_sched_barrier(0);
    });
    return acc;
}

// As a function of its own, so that its rows cost the kernel no registers.
__device__ __noinline__ uint32_t find_verdict_apart(uint64_t* word, uint64_t epoch, const uint32_t* want, uint32_t affine,
                                                    const FF_LDS u32x4* weight, const uint8_t* at, uint32_t n,
                                                    uint32_t lane_c, int lane)
{
    return find_verdict<kBlockRows>(word, epoch, want, affine, weight, at, n, lane_c, lane);
}

// 16 bytes of the stream at pos to wherever they belong, by a lane on its own.
__device__ __noinline__ void scatter_slot(const uint64_t* __restrict__ seg_off, const uint64_t* __restrict__ seg_ptr,
                                          uint32_t first, uint32_t last, uint64_t pos, uint64_t payload, u32x4 w)
{
    if (pos >= payload) return;
    while (first < last) {
        const uint32_t mid = first + (last - first + 1) / 2;
        if (seg_off[mid] <= pos) first = mid; else last = mid - 1;
    }
    uint64_t a = seg_off[first], b = seg_off[first + 1], base = seg_ptr[first];
    if (pos + 16 <= b) {
        store16_unaligned(reinterpret_cast<uint8_t*>(base + (pos - a)), w);
        return;
    }
    const uint32_t d[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int u = 0; u < 8; u++) {
        const uint64_t p = pos + 2u * u;
        if (p >= payload) return;
        while (p >= b) {
            first++;
            a = b;
            b = seg_off[first + 1];
            base = seg_ptr[first];
        }
        *as_global(reinterpret_cast<uint16_t*>(base + (p - a))) = static_cast<uint16_t>(d[u >> 1] >> ((u & 1) * 16));
    }
}

// All rows of a tile so, read from the buffer; bp: the lane's slot of row 0 there.
__device__ __forceinline__ void scatter_slots(const uint64_t* __restrict__ seg_off, const uint64_t* __restrict__ seg_ptr,
                                              const uint32_t* __restrict__ tile_first_seg, const TileTables& T,
                                              const uint32_t tile, const uint8_t* bp, const int lane)
{
    const uint32_t first = tile_first_seg[tile];
    const uint32_t last = tile + 1 < T.n_tiles ? tile_first_seg[tile + 1] : T.n_seg - 1;
#pragma unroll 1
    for (uint32_t r = 0; r < kRows; r++)
        scatter_slot(seg_off, seg_ptr, first, last, static_cast<uint64_t>(tile) * kTileBytes + r * kRowBytes + 16u * lane,
                     T.payload, load16_stream<false>(bp + r * kRowBytes));
}

// The tile's rows to their tensors.  A tile inside one tensor goes out as it is if it starts on a 128-byte
// line there, else shifted through a two-row ring in LDS so that all but the edges of its stores lie on lines
// (as the tile kernel's restore does); up to four tensors: every lane picks its own by comparing its
// place with the boundaries; more: slot by slot, read again.
template <bool SEG_NT>
__device__ __forceinline__ void scatter_tile(const uint64_t* __restrict__ seg_off,
                                             const uint64_t* __restrict__ seg_ptr,
                                             const uint32_t* __restrict__ tile_first_seg, const TileTables& T,
                                             const uint32_t tile, const uint64_t base,
                                             const uint8_t* bp, const u32x4 (&w)[kRows], uint32_t* ring, const int lane)
{
    const uint32_t lane16 = 16u * lane;
    const uint64_t s = static_cast<uint64_t>(tile) * kTileBytes;
    if (base && (base & 127u) == 0) {
        uint8_t* const tp = reinterpret_cast<uint8_t*>(base) + lane16;
        static_for<kRows>([&](auto r) { store16_unaligned<SEG_NT>(tp + r * kRowBytes, w[r]); });
        return;
    }
    if (base) {
        const uint32_t m = static_cast<uint32_t>(base) & 127u;
        uint8_t* const ap = reinterpret_cast<uint8_t*>(base - m) + lane16;  // lane's slot, output row 0
        // rows lie at byte 1024 * (row & 1); bytes [2048, 2064) repeat bytes [0, 16)
        const uint32_t o0 = (lane16 - m) & 2047u, o1 = (o0 + 1024u) & 2047u, sh = (m & 2u) * 8u;
        const uint32_t* const r0 = ring + (o0 >> 2);
        const uint32_t* const r1 = ring + (o1 >> 2);
        auto take = [&](const uint32_t* r) {
            uint32_t d[5];
            static_for<5>([&](auto k) { d[k] = r[k]; });
            return u32x4{__builtin_amdgcn_alignbit(d[1], d[0], sh), __builtin_amdgcn_alignbit(d[2], d[1], sh),
                         __builtin_amdgcn_alignbit(d[3], d[2], sh), __builtin_amdgcn_alignbit(d[4], d[3], sh)};
        };
        auto store_part = [&](uint8_t* p, const u32x4 y, const uint32_t lo, const uint32_t hi) {
            if (lane16 >= lo && lane16 + 16u <= hi) {
                store16_stream<SEG_NT>(p, y);
            } else if (lane16 + 16u > lo && lane16 < hi) {
                const uint32_t d[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
                for (int u = 0; u < 8; u++) {
                    const uint32_t pos = lane16 + 2u * u;
                    if (pos >= lo && pos < hi)
                        *as_global(reinterpret_cast<uint16_t*>(p + 2 * u)) =
                            static_cast<uint16_t>(d[u >> 1] >> ((u & 1) * 16));
                }
            }
        };
        static_for<kRows>([&](auto J) {
            *reinterpret_cast<u32x4*>(ring + (J & 1) * 256 + 4 * lane) = w[J];
            if ((J & 1) == 0 && lane == 0) *reinterpret_cast<u32x4*>(ring + 512) = w[J];
            const u32x4 y = take((J & 1) ? r1 : r0);
            if (J == 0)
                store_part(ap, y, m, kRowBytes);
            else
                store16_stream<SEG_NT>(ap + J * kRowBytes, y);
            __builtin_amdgcn_sched_barrier(0);
        });
        store_part(ap + kRows * kRowBytes, take(r0), 0u, m);
        return;
    }
    if (s >= T.payload) return;
    const uint32_t first = tile_first_seg[tile];
    auto seg_begin = [&](uint32_t k) { return seg_off[first + k < T.n_seg ? first + k : T.n_seg]; };
    const uint64_t a0 = seg_begin(0), a1 = seg_begin(1), a2 = seg_begin(2), a3 = seg_begin(3), a4 = seg_begin(4);
    if (a4 >= s + kTileBytes || a4 >= T.payload) {
        const uint64_t left = T.payload - s;
        const uint32_t end = left < kTileBytes ? static_cast<uint32_t>(left) : kTileBytes;
        // address of the tile's byte 0 if it were in that tensor, and the boundaries relative to the tile
        auto seg_base = [&](uint32_t k, uint64_t a) {
            return seg_ptr[first + k < T.n_seg ? first + k : T.n_seg - 1] + (s - a);
        };
        auto bound = [&](uint64_t a) { return a - s < kTileBytes ? static_cast<uint32_t>(a - s) : kTileBytes; };
        const uint64_t b0 = seg_base(0, a0), b1 = seg_base(1, a1), b2 = seg_base(2, a2), b3 = seg_base(3, a3);
        const uint32_t c0 = bound(a1), c1 = bound(a2), c2 = bound(a3);
        const uint64_t step1 = b1 - b0, step2 = b2 - b1, step3 = b3 - b2;
        auto place = [&](uint32_t rel) {
            return b0 + (rel >= c0 ? step1 : 0) + (rel >= c1 ? step2 : 0) + (rel >= c2 ? step3 : 0) + rel;
        };
        static_for<kRows>([&](auto J) {
            const uint32_t rel = J * kRowBytes + lane16;
            const bool straddle = (rel < end && rel + 16u > end) || (rel < c0 && rel + 16u > c0) ||
                                  (rel < c1 && rel + 16u > c1) || (rel < c2 && rel + 16u > c2);
            if (rel < end && !straddle) {
                store16_unaligned<SEG_NT>(reinterpret_cast<uint8_t*>(place(rel)), w[J]);
            } else if (rel < end) {
                const uint32_t d[4] = {w[J].x, w[J].y, w[J].z, w[J].w};
#pragma unroll
                for (int u = 0; u < 8; u++)
                    if (rel + 2u * u < end)
                        *as_global(reinterpret_cast<uint16_t*>(place(rel + 2u * u))) =
                            static_cast<uint16_t>(d[u >> 1] >> ((u & 1) * 16));
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        return;
    }
    scatter_slots(seg_off, seg_ptr, tile_first_seg, T, tile, bp, lane);
}

// (The tables as pointers of their own: what is read through them is then known not to change, and comes by
// scalar loads, which no wait for the rows has to wait for.)
template <int HINT>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(3))) void tile_kernel_held(
    const uint64_t* __restrict__ seg_off, const uint64_t* __restrict__ seg_ptr,
    const uint32_t* __restrict__ tile_first_seg, const uint64_t* __restrict__ tile_base,
    const uint32_t* __restrict__ tile_shift, TileTables T, const uint8_t* __restrict__ chunks)
{
    constexpr bool kSegNT = (HINT & 1) != 0, kBufNT = (HINT & 2) != 0;
    const uint32_t block = block_behind_args<0, 5 * sizeof(void*) + sizeof(TileTables) + sizeof(void*) + 4>();
    __shared__ HoldLds lds;
    const int lane = threadIdx.x & (kWaveSize - 1);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWaveSize);
    table_to_lds<kThreads, sizeof(lds.weight)>(T.block_tab, &lds.weight[0][0], wave, lane);
    if (threadIdx.x < kWaves) lds.sum[threadIdx.x] = lds.verdict[threadIdx.x] = 0;
    __builtin_amdgcn_sched_barrier(0);
    const uint32_t tile = xcd_order(block, gridDim.x, T.xcd_group) * kWaves + wave;
    if (tile >= T.n_tiles) {
        wait_loads<0>();
        workgroup_barrier();
        return;
    }
    // the lane's factors in the four blocks, the tile's distance to the end of its chunk
    const uint32_t* const lane_tab = T.block_tab + kBlockRows * 4 * kWeightWords + lane;
    uint32_t c[kBlocks];
    static_for<kBlocks>([&](auto b) { c[b] = lane_tab[(kBlocks - 1 - b) * kWaveSize]; });
    const uint32_t in_chunk = tile & (T.tiles_per_chunk - 1), chunk = tile >> T.tpc_log2;
    const uint32_t shift = tile_shift[in_chunk];
    const uint64_t base = tile_base[tile];
    const uint32_t want = table_entry(T.want, chunk);
    const uint8_t* const bp = chunks + static_cast<uint64_t>(tile) * kTileBytes + 16u * lane;
    u32x4 w[kRows];
    static_for<kRows>([&](auto r) { w[r] = load16_stream<kBufNT>(bp + r * kRowBytes); });
    wait_loads<kRows>();  // for the weights; the rows are behind them
    workgroup_barrier();
    uint32_t x = 0;
    static_for<kBlocks>([&](auto b) {
        const f32x16 acc = block_sums(lds, lane, [&](auto r) { return w[b * kBlockRows + r]; });
        x ^= gf2_mul_half(matrix_halves(acc), c[b]);
    });
    uint32_t reg = gf2_mul(wave_xor(x), shift);
    // the wavefronts of this workgroup that are at the same chunk: the last one goes to the tally, and waits
    // for the chunk's verdict on behalf of the others
    const uint32_t run = T.tiles_per_chunk < uint32_t(kWaves) ? T.tiles_per_chunk : uint32_t(kWaves);
    const uint32_t lead = wave - (wave & (run - 1));
    uint32_t speaks = 0;
    if (lane == 0 && (run == 1 || run_complete(lds.sum[lead], wave - lead, run, reg))) {
        tally_run<kRestore>(T, reg, chunk, in_chunk / run, T.tiles_per_chunk / run, chunk, T.n_chunks, want);
        speaks = 1;
    }
    volatile uint32_t* const said = &lds.verdict[lead];
    uint32_t verdict = 0;
    if (__builtin_amdgcn_readfirstlane(speaks)) {
        verdict = await_verdict(T, chunk);
        if (!verdict) {  // alone, and with rows read again: this rare case would need the registers of both
            const uint32_t n = T.tiles_per_chunk * kBlocks;
            verdict = __builtin_amdgcn_readfirstlane(find_verdict_apart(
                T.verdict + chunk, T.epoch, T.want + chunk, T.affine, (const FF_LDS u32x4*)&lds.weight[0][0],
                chunks + static_cast<uint64_t>(chunk) * n * kBlockBytes, n, c[kBlocks - 1], lane));
            *said = verdict;
            if (verdict == 2) scatter_slots(seg_off, seg_ptr, tile_first_seg, T, tile, bp, lane);
            return;
        }
        *said = verdict;
    } else {
        while (!(verdict = __builtin_amdgcn_readfirstlane(*said))) __builtin_amdgcn_s_sleep(2);
    }
    if (verdict == 3) return;
    scatter_tile<kSegNT>(seg_off, seg_ptr, tile_first_seg, T, tile, base, bp, w, lds.ring[wave], lane);
}

}  // namespace hold

}  // namespace ffsnap
