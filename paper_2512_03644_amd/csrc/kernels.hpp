// Launch wrappers of the GPU kernels (kernels.hip).  Every wrapper enqueues on `stream`,
// returns hipSuccess or the launch error, and never synchronises.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "xcd_order.h"

namespace ffsnap {

// Run length of the XCD-aware workgroup order (xcd_order.h) of the kernels that move 32 KiB per
// wavefront, 128 KiB per workgroup.
constexpr uint32_t kDefaultXcdGroup = 2048;

// Restores, and packs in blocks, of more than kShortRunsFrom bytes take short runs instead, in tiles of 1 MB, in blocks of 512 KB
// (of 1 MB above kLongerRunsFrom), so that the XCDs sweep one region and not eight.  Default / short, us: pack of 75 / 90 / 100 / 130 /
// 180 MB 24.9 / 32.6 / 45.4 / 54.1 / 74.3 and 25.1 / 31.2 / 41.8 / 50.9 / 70.7, of 5 KiB tensors 0.15 / 0.3 / 1 GB 61.9 / 113.8 /
// 356.8 and 59.4 / 110.6 / 348.4; restore of 60 / 110 / 150 / 300 / 600 MB 22.7 / 44.8 / 60.7 / 123.3 / 223 and 22.8 / 42.6 / 56.5 /
// 116.2 / 213, of 1 / 2 / 4 GB 354 / 667 / 1345 and 342 / 650 / 1334, 11.8 GB 3642 both; of 5 KiB tensors 0.3 / 1 GB 121.6 / 407.1 and
// 116.5 / 402.7; 24 listed chunks of them 44.3 and 43.5.  A pack on tiles gains or loses as the tensors lie (0.3 / 0.6 GB 117.6 / 222.9
// and 115.2 / 213.2, of large tensors in one allocation 112.2 / 207.8 and 120.9 / 215.0; 15 GB 4862 and 4928), a verify nothing.
// First passes over new states (medians of 9 to 20) gain as well or lose nothing, the code with long runs alone / with short ones:
// restore of 110 / 300 MB, 1 / 3 GB 68.7 / 151.4 / 391.6 / 1078 and 63.7 / 142.6 / 376.8 / 1069, of 5 KiB tensors,
// 0.15 / 0.3 GB 86.9 / 148.3 and 80.6 / 136.6, pack of 130 MB 76.7 and 75.1, of 5 KiB tensors, 0.3 GB 189.2 and 178.0; by run length alone,
// 8 / 16 / 32 / 64 / 128 / 512 / 2048, restore of 5 KiB tensors, 1 GB 439 / 434 / 440 / 435 / 441 / 437 / 439, 28 listed chunks of 4 MiB
// 137 / 134 / 128 / 128 / 132 / 136 / 136 (these differ by 8 between states).
constexpr uint32_t kShortXcdGroup = 8;
constexpr uint64_t kShortRunsFrom = 80ull << 20, kLongerRunsFrom = 384ull << 20, kShortRunsTo = 4096ull << 20;

constexpr uint32_t kTallyFan = 32;
// A verdict on more chunks than this does without the tally: the returning atomics of a chunk hold its
// workgroup up, and the last level counts a word per 32 chunks on one address, which the two launches that
// the tally saves no longer pay for.  With it / without, us (blocks with byte tables): 4096 chunks (64 MB) restore 27.6 / 28.1, verify
// 18.8 / 21.3; 6080 (190 MB) 75.6 / 77.7, 41.1 / 41.6; 8000 (1 GB) 338.6 / 337.5, 166.1 / 164.2; 8192 (64 MB)
// 31.0 / 28.1, 22.5 / 21.3; 64000 (1 GB) 476.8 / 464.1, 316 / 300.
constexpr uint64_t kTallyChunks = 6144;
// Verdicts on so many chunks in blocks are not counted one by one, level above level at 0.7 us each: the damaged ones
// alone are (7 chunks 6.7 us with the count, 6.0 without; 78 chunks 12.0 and 10.8).  On more chunks a buffer that is
// damaged all over would be bound by the one word that they are counted on, at 50 ns each.
constexpr uint32_t kDirectChunks = 128;
// Words of a plan's tally (0: none), enough for runs of 8 blocks of 8 KiB and of 4 tiles of the plan's size
// or more.  None if its chunks have more runs than there are levels for, or its tiles are smaller than a
// block: those are bound by what a tile costs beyond its bytes, and a returning atomic each is too much
// of it (restore of 4 MB in chunks of 4 KiB 15.8 us with, 14.0 without; 64 MB 80.2 / 74.7).
inline uint64_t tally_size(uint64_t n_chunks, uint64_t chunk_bytes, uint64_t tile_bytes)
{
    if (tile_bytes < (1ull << 13)) return 0;
    const uint64_t run = 4 * tile_bytes < (8ull << 13) ? 4 * tile_bytes : (8ull << 13);
    const uint64_t runs = chunk_bytes > run ? chunk_bytes / run : 1;
    if (runs > kTallyFan * kTallyFan) return 0;
    return 1 + (n_chunks + kTallyFan - 1) / kTallyFan + n_chunks + (runs > kTallyFan ? n_chunks * (runs / kTallyFan) : 0);
}

// Device-side view of a plan's tables, plus the constants the tile kernels need.
struct TileTables {
    const uint64_t* seg_off = nullptr;        // [n_seg + 1] stream offsets, seg_off[n_seg] = payload
    const uint64_t* seg_ptr = nullptr;        // [n_seg] device addresses
    const uint32_t* tile_first_seg = nullptr; // [n_tiles]
    const uint64_t* tile_base = nullptr;      // [n_tiles] tensor-side address of a tile that lies
                                              // inside one segment, else 0 (may be absent)
    const uint32_t* block_tab = nullptr;      // tables of the 8 KiB blocks (build_block_tab)
    const uint32_t* run_tab = nullptr;        // [runs of 8 blocks in a chunk][32]: what bit i of a run's register
                                              // is at the end of the chunk (build_run_tab)
    const uint32_t* tab_u = nullptr;          // [4][256] multiply-by-x^8192 byte tables, then
                                              // [64] lane constants x^(128 * (63 - lane))
    // Where a tile's register goes.  acc set: XORed (atomically) into acc[chunk of the tile], an
    // array of the caller that launch_preset has prepared; nothing else is written, so calls that
    // share these tables may overlap in time.  Else partial set: stored to partial[tile] (a
    // buffer CRC over caller-provided scratch).  Neither: the pass only moves bytes.
    uint32_t* acc = nullptr;
    uint32_t* partial = nullptr;
    // If tally is set (all zero before and after every call; one call at a time), acc[]
    // gets the results themselves -- the CRC32C (pack), or 0 / 1 by comparison with want[] and *n_bad
    // the number of ones (plus what it held, with n_bad_add) -- and no kernel before or after is
    // needed.  Its words: [1] all chunks, [ceil(n_chunks / kTallyFan)] groups of chunks, [n_chunks]
    // chunks, and if a chunk has more than kTallyFan runs -- the tiles or blocks of a chunk that one
    // workgroup takes -- [n_chunks][runs / kTallyFan].
    uint32_t block_log2 = 0;  // blocks: the tables' tiles hold 2^block_log2 of them
    uint64_t* tally = nullptr;
    const uint32_t* want = nullptr;
    uint64_t* n_bad = nullptr;
    uint32_t n_bad_add = 0;
    // The call's number in the plan, from 1: no two calls have the same, so what is marked with it is never set back.
    // Who waits for verdicts (hold.h) finds them in verdict, [n_chunks] of the plan's own words (verdict_word).
    uint64_t epoch = 0;
    uint64_t* verdict = nullptr;
    // Verdicts without the levels of the tally above its chunks (open_count in tally.h); state: a word of the
    // plan's, 2 * epoch and more from when *n_bad is being set to zero.
    uint64_t* state = nullptr;
    uint32_t direct = 0;
    uint32_t polls = 0;       // how often one looks before it finds the verdict by itself
    uint32_t affine = 0;      // preset/complement term of a chunk
    uint32_t n_chunks = 0;
    // If set: [plan tiles per chunk] x^(32 + 8 * bytes from the end of tile k of a chunk to the
    // end of the chunk).  A tile's register, which lacks the factor x^32 of a CRC register, is
    // multiplied by its entry, so that the registers of a chunk combine by XOR alone.  A pass
    // that folds groups of shift_stride plan tiles as one uses the entry of the group's last tile.
    const uint32_t* tile_shift = nullptr;
    uint32_t shift_stride = 1;
    uint64_t payload = 0;                     // N
    uint64_t total_rows = 0;                  // 1 KiB rows in the buffer
    uint32_t n_seg = 0;
    uint32_t tile_rows = 0;                   // rows per tile
    uint32_t lead_rows = 0;                   // rows missing at the front of tile 0
    uint32_t n_tiles = 0;
    uint32_t hint = 3;                        // bit 0: non-temporal tensor-side accesses, bit 1: buffer-side
    uint32_t n_list = 0;                      // > 0 selects tiles [tile_begin, tile_begin + n_list)
    uint32_t tile_begin = 0;
    const uint32_t* skip_bad = nullptr;       // if set: bad[] per chunk; tiles of bad chunks are left out
    uint32_t tiles_per_chunk = 1;             // of this pass (a power of two) ...
    uint32_t tpc_log2 = 0;                    // ... and its logarithm
    // Workgroups are dealt to the 8 XCDs round-robin.  With xcd_group = G > 0 the workgroups of
    // one XCD take G consecutive groups of tiles, the next XCD the following G, and so on, so
    // that every XCD (and its L2) sweeps runs of G * 128 KiB instead of every eighth 128 KiB.
    uint32_t xcd_group = kDefaultXcdGroup;  // measured: 8 .. 2048 within 0.5 % on a 12 GB shard, 2048 best
                                // (by 1-2 %) on a 15 GB one; 0 (launch order) costs 5-7 %
};

// What the word of a chunk holds when the call has found it sound (0) or damaged (1).  The whole number: calls
// that write no verdicts, and those are most, count as well, so a word may be as old as the plan.
__host__ __device__ inline uint64_t verdict_word(uint64_t epoch, uint32_t bad) { return epoch << 1 | bad; }

enum TileMode { kPack = 0, kRestore = 1, kVerify = 2 };

// The cache hint of a pass over a buffer small enough to be still in the 256 MiB last-level cache, from
// where it was written or received: plain loads, non-temporal stores.
constexpr uint32_t kHintWarm(TileMode mode) { return mode == kPack ? 2u : 1u; }

// A list of chunks handed to a kernel by value, inside its arguments: a selective restore needs
// no device memory of its own for it.  Longer lists are processed in several launches.
constexpr uint32_t kMaxListedChunks = 254;
struct ChunkList {
    uint32_t n = 0;
    uint32_t id[kMaxListedChunks];
};

// Folds every tile: kPack gathers segments -> chunks; kRestore reads chunks and scatters to the
// segments; kVerify only reads chunks.  With `list` (kRestore / kVerify, registers into t.acc)
// only the tiles of the listed chunks are processed.
hipError_t launch_tiles(TileMode mode, const TileTables& t, void* chunks, hipStream_t stream,
                        const ChunkList* list = nullptr);

// The same in blocks of kBlockBytes, one wavefront each (blocks.hip): what launch_tiles does for
// tables whose tiles have that size.  as_blocks() makes such tables of a plan's with larger tiles, up
// to the 8 blocks of a run: run_tab knows the ends of runs of that size.
constexpr uint32_t kBlockBytes = 8192;
constexpr uint32_t kMaxBlockTileBytes = 8 * kBlockBytes;
hipError_t launch_blocks(TileMode mode, const TileTables& t, void* chunks, hipStream_t stream,
                         const ChunkList* list);
inline TileTables as_blocks(TileTables t)
{
    for (; t.tile_rows > kBlockBytes / 1024; t.tile_rows /= 2) {
        t.block_log2++;
        t.n_tiles *= 2;
        t.tiles_per_chunk *= 2;
        t.tpc_log2++;
    }
    return t;
}
inline bool tiles_are_blocks(const TileTables& t)
{
    // (tiles grouped for a read-only pass may be as long, but their shifts lie shift_stride apart)
    return t.tile_rows == kBlockBytes / 1024 && t.shift_stride == 1 && t.block_tab && !t.partial;
}

// Verifies every chunk and scatters those that verify, reading the buffer once: tables with tiles of 32 KiB
// (hold.h) or of blocks (blocks.hip), T.acc, T.tally, T.verdict.  A wavefront keeps its tile until its chunk's
// verdict is there, so the workgroups of a chunk should be in flight together: in runs of kHoldXcdGroup
// workgroups an XCD (3.2 GB of 20,000 ragged tensors 1190 / 1179 / 1185 / 1248 us with runs of 1 / 8 / 16 / 32, of
// 3.3 GB in chunks of 8 MiB 1145 / 1131 / 1207 with 4 / 8 / 16), and no more than a third (blocks: half) of
// what the chip holds.  Against two passes, us: chunks of 256 KiB 1510 / 1096, 4 MiB 1524 / 1155, 32 MiB 1545 / 1191;
// ragged in chunks of 32 KiB 1632 / 1188, 4 MiB 1572 / 1184; 4 / 16 / 64 / 100 / 180 MB 15.8 / 18.5 / 40.9 / 55.9 / 100
// and 9.2 / 12.0 / 28.6 / 47.0 / 72; small tensors 60 / 150 / 1000 MB 45.9 / 99 / 544 and 37.9 / 97 / 492.
constexpr uint32_t kHoldXcdGroup = 8, kHoldPolls = 4096;
inline uint64_t hold_chunk_bytes(const TileTables& t, uint64_t compute_units)
{
    return compute_units * (tiles_are_blocks(t) ? 8 * kBlockBytes : 128u << 10);  // 256: 16 and 32 MiB
}
hipError_t launch_held(const TileTables& t, void* chunks, hipStream_t stream);

// Fills tab (host, kBlockTabWords entries): the weights of the 32 dwords of a lane (matrix_fold.h), then
// for k = 0..7 and every lane its factor for the place of its column in a row, plus k blocks, and the same
// plus half a block.
constexpr int kBlockTabWords = 32 * 4 * 64 + 2 * 8 * 64;
constexpr uint64_t kLeanBlocks = 16384;  // packs of more blocks take half the weights (block_kernel_lean)
void build_block_tab(uint32_t* tab);

// Fills tab (host): for the k-th of `runs` runs of run_bytes bytes of a chunk, words 32 k + i = x^(31 - i) *
// x^(32 + 8 * bytes from the run's end to the chunk's).  A run's register is one lane's, and a product of 32
// dependent steps took it 0.5-0.7 us at the end of every small call; with its bits spread over the lanes it is one
// word each and an XOR over the lanes (pack / restore of 32 MB 15.5 / 16.0 -> 14.9 / 15.3 us, verify of 3.2 MB 7.2 ->
// 6.7).
void build_run_tab(uint32_t* tab, uint64_t runs, uint64_t run_bytes);

// out[j] = affine (crcs null: pack) or affine ^ crcs[j] (verify) for chunks [first, first + n), or
// for the listed chunks; *n_bad = 0 if n_bad is not null.  The tiles then XOR their registers in.
hipError_t launch_preset(uint32_t* out, const uint32_t* crcs, uint64_t first, uint64_t n,
                         uint32_t affine, uint64_t* n_bad, const ChunkList* list,
                         hipStream_t stream);

// bad[j] = (bad[j] != 0) for chunks [0, n), or for the listed chunks; *n_bad += their number.
hipError_t launch_finish_verify(uint32_t* bad, uint64_t n, uint64_t* n_bad, const ChunkList* list,
                                hipStream_t stream);

// CRC of one buffer: combine n_tiles registers, then run the register over `tail_bytes` more
// bytes at `tail`, then apply the preset/complement term `affine`.
hipError_t launch_finish_crc(const uint32_t* partial, uint32_t n_tiles, uint32_t x_tile,
                             const uint8_t* tail, uint32_t tail_bytes, uint32_t affine,
                             uint32_t* out, hipStream_t stream);

// Verify pass over every chunk of a buffer with one workgroup per chunk (no atomics on the
// per-chunk words, no preset, no finish): sets *n_bad = 0, then bad[j] and *n_bad.  Usable when
// verify_chunks_applicable(); t supplies the tables (tile_shift for the plan's own tile size).
bool verify_chunks_applicable(uint64_t chunk_bytes, uint64_t n_chunks);
hipError_t launch_verify_chunks(const TileTables& t, uint64_t chunk_bytes, uint32_t tile_bytes,
                                uint32_t plan_tiles_per_chunk, uint32_t affine, const void* chunks,
                                const uint32_t* crcs, uint32_t* bad, uint64_t* n_bad,
                                uint64_t n_chunks, hipStream_t stream);

hipError_t launch_zero_u64(uint64_t* p, hipStream_t stream);

hipError_t launch_copy(void* dst, const void* src, uint64_t nbytes, hipStream_t stream);

// Fills tab (host, kTabWords entries): byte tables of multiplication by x^8192, then the 64 lane
// constants x^(128 * (63 - lane)).
constexpr int kTabWords = 1024 + 64;
void build_tab_u(uint32_t* tab);

}  // namespace ffsnap
