// Host-side layout of a snapshot: validation of the segment list, stream offsets, parameter
// groups, tiling.  No GPU calls in here.
#pragma once
#include <stdint.h>

#include <vector>

#include "../../include/ffsnap.h"

namespace ffsnap {

struct Seg {
    uint64_t ptr;     // device address
    uint64_t off;     // stream offset of the first byte
    uint64_t nbytes;  // > 0
    uint32_t dtype, kind, param_id;
};

struct Param {
    uint32_t param_id;
    int32_t seg[4];   // indices into Layout::segs for W16, MASTER, M, V (-1 = missing)
    uint64_t numel;
};

struct Layout {
    uint64_t chunk_bytes = 0, payload = 0, n_chunks = 0, buffer_bytes = 0;
    std::vector<Seg> segs;      // non-empty segments, stream order
    std::vector<Param> params;  // ascending param_id
    bool adam_ok = false;       // every non-RAW segment belongs to a complete, consistent group
    uint32_t half_dtype = 0;    // format of the working weights: FF_BF16 or FF_F16 (0: no groups)
    uint32_t layout_id = 0;
    // tiling: a tile is the stream range one wavefront folds; it never crosses a chunk
    uint64_t tile_bytes = 0, n_tiles = 0;
    uint32_t tiles_per_chunk = 0;
    std::vector<uint32_t> tile_first_seg;  // segment holding the first byte of each tile
                                           // (segs.size()-1 for tiles past the payload)
    // Tensor-side address of a tile's first byte if the whole tile lies inside one segment, else
    // 0: lets a wavefront start such a tile after one table read instead of a walk through the
    // segment tables.
    std::vector<uint64_t> tile_base;
};

// Unit of work of the fused optimizer step: the elements of one parameter group (its four streams
// w16/master/m/v) that lie in one aligned block of kParamTileElems elements, or the bytes of a RAW
// segment that lie in one aligned block of kRawTileBytes bytes of the stream.  A block is cut wherever
// one of its streams crosses a chunk boundary, so each stream of a tile lies inside one chunk and
// adds one term ("piece") to that chunk's CRC.  Tiles are aligned to the tensors' elements rather
// than to the cuts, so that behind a cut the rows go on where the tensors' memory lines lie.
// A tile's register is taken over the whole block, with zeros where the block is not the tile's;
// zeros in front do not change a register started from 0 and zeros behind multiply it by a power of
// x, so shift = x^(32 + 8 * bytes from the END OF THE BLOCK to the end of the chunk), an exponent
// that may be negative.  (The register lacks the factor x^32 that a CRC register carries.)
// An fp32 element that straddles a chunk boundary (its stream offset is 2 mod 4) starts a tile; its
// first two bytes form a separate "head" piece that ends the previous chunk.
struct WorkTile {
    uint64_t ptr[4];    // addresses of the tile's first element: w16, master, m, v (RAW: ptr[0])
    uint64_t soff[4];   // stream offsets of the tile's first byte in each stream
    uint32_t chunk[7];  // pieces 0..3: the four streams; 4..6: head pieces of master, m, v
    uint32_t shift[7];  // see above; head pieces: 1; 0 = piece absent
    uint64_t e0;        // first element within the parameter (indexes the gradient)
    uint32_t n;         // elements (parameter tile) or bytes (RAW tile)
    uint32_t kind;      // 0 = parameter group, 1 = RAW
    uint32_t grad_index;
    uint32_t head_split;  // bit x set: the first element of stream x is split as described
};

constexpr uint32_t kWorkParam = 0, kWorkRaw = 1;
constexpr uint32_t kParamTileElems = 1u << 13;
constexpr uint32_t kRawTileBytes = 1u << 15;

// What one wavefront of the fused step works on: one sub-block of a tile.  kWavesPerGroup
// consecutive entries make a workgroup; the entries of a run, all in one workgroup, sum their registers in
// LDS before they go to memory.  A run is the entries of one parameter tile; or, as RAW tiles lie in
// stream order and have one stream, the neighbouring entries of all RAW tiles in one chunk.
struct WorkWave {
    uint32_t tile;  // index into the tile list, or kNoTile: nothing to do
    uint32_t info;  // bits 0..3 sub-block of the tile's block, 4..6 place of the run's first
                    // wavefront in the workgroup, 8..11 wavefronts in the run, 16..31 of a parameter tile
                    // the group's number in its launch
};
constexpr uint32_t kNoTile = 0xFFFFFFFFu;
constexpr uint32_t kWavesPerGroup = 8;
constexpr uint32_t kSubElems = kParamTileElems / 16; // 2 rows of 256 elements
constexpr uint32_t kSubRawBytes = kRawTileBytes / 4; // 8 rows of 1 KiB

// Work list of the fused step over the whole layout (needs L.adam_ok): the parameter tiles first,
// then the RAW tiles.
void build_work_tiles(const Layout& L, std::vector<WorkTile>& out);

// The wavefronts of the tiles, launch by launch: launch k takes the parameter groups
// [k * groups_per_launch, (k + 1) * groups_per_launch), the last launch the RAW tiles as well.
// begin[k] is the first entry of launch k, one more entry the end; each a multiple of
// kWavesPerGroup.  groups_per_launch <= 65536.  False, with out and begin unfinished, if there would be more than max_entries: the
// kernels count tiles and entries in 32 bits, and a tile has up to 16 entries.
constexpr uint64_t kMaxWorkEntries = 0xFFFFFFF0ull;
bool build_work_waves(const std::vector<WorkTile>& tiles, uint64_t n_params,
                      uint32_t groups_per_launch, std::vector<WorkWave>& out,
                      std::vector<uint32_t>& begin, uint64_t max_entries = kMaxWorkEntries);

// Where a contribution to a chunk's checksum goes in a step that sums them up in 64-bit words (tally.h): leaf words of
// up to 32 contributions each, and above a chunk's leaves, if there are several, a root.
struct StepTicket {
    uint32_t leaf, leaf_full;  // the word, and its upper half when everything is there
    uint32_t bits;             // bits 0..4 the contribution's bit in it, 8..13 leaves of the chunk, 16..20 the leaf's bit in the root
    uint32_t root;             // the word above, if there are several leaves
};
// Contributions of the step with these work lists: for every wavefront entry that begins a run four tickets (streams
// 0 to 3; the first alone if all streams are in one chunk, or for RAW), for every tile three (its head pieces, streams
// 1 to 3), others left at zero.  words: how many words there are.  False if a chunk has more than 1024 contributions.
bool build_step_tickets(const std::vector<WorkTile>& tiles, const std::vector<WorkWave>& waves, uint64_t n_chunks,
                        std::vector<StepTicket>& runs, std::vector<StepTicket>& heads, uint64_t& words);

// Do most elements of these parameter tiles have an fp32 stream, in place or in the snapshot, whose rows lie
// off its 128-byte lines?  (A buffer that is itself on a line is assumed.)
bool mostly_off_lines(const WorkTile* tiles, uint64_t n);

// Returns FF_OK or a negative ff_status; `out` is valid only on FF_OK.
// tile_log2: 0 = default tile size, else log2 of the tile size in bytes (clamped to
// [10, log2(chunk_bytes)]).
int build_layout(const ff_segment* segs, uint64_t n_segs, uint64_t chunk_bytes, unsigned tile_log2,
                 Layout& out);

// Tile size when the caller names none.  32 KiB tiles keep the region the chip is sweeping at any
// moment compact, which is what a pass that reads and writes needs; a read-only pass amortises the
// per-tile reduction better on 64 KiB.  Tiles of 8 KiB (blocks, blocks.hip) are for two kinds of plan.
// Small buffers, where 32 KiB per wavefront leaves the chip idle and launches count.  Three buffers in turn,
// tensors on 128-byte lines, 32 KiB tiles against blocks, us: pack of 32 / 64 / 96 / 112 / 128 / 160 / 190 MB
// 20.2 / 30.8 / 41.8 / 48.8 / 53.0 / 63.0 / 73.2 against 15.4 / 25.7 / 40.7 / 47.1 / 53.4 / 64.7 / 75.6, restore of
// 96 / 112 / 128 / 190 MB 44.4 / 52.0 / 55.9 / 76.6 against 41.4 / 49.4 / 55.5 / 78.1 (on a stream without the
// tally blocks take 1-2 us more).  Where most tiles are off the lines or hold a boundary blocks win for longer:
// tensors 6 bytes off a line, restore of 128 / 160 / 190 MB 66.3 / 76.5 / 87.0 against 59.5 / 70.9 / 82.3,
// pack 62.2 / 67.8 / 78.3 against 59.4 / 67.8 / 78.3; 300 ragged tensors in 186 MB 82.8 against 78.1 (pack); and
// so they do where a chunk leaves no room for a 32 KiB tile.  A read-only pass is as fast or faster in
// blocks up to there on any layout (verify of 96 / 128 / 144 / 160 / 190 MB 27.8 / 30.5 / 38.6 / 39.6 / 42.8
// against 24.9 / 29.9 / 32.8 / 36.8 / 41.0).  And lists of small tensors, whose tiles of more
// than four tensors take the tile kernel's row-by-row path: 5 KiB tensors (1 GB) 890 and 373 us; tensors
// of 40 KB on average (0.8 GB) 302 and 291 us.  With 110 KB it is 318 and 312 for a pack but 459 and 483
// for a restore that leaves bad chunks out: too few of those tiles are crowded.
// (All of this with byte tables in LDS in the blocks, before the matrix product.  With it blocks lead further up: tensors
// on the lines, tiles / blocks, pack of 128 / 160 / 192 / 256 / 400 MB 66.4 / 68.2 / 82.8 / 100.5 / 142 against 49.8 / 62.1 /
// 72.6 / 93.9 / 139, restore 55.7 / 67.6 / 77.1 / 97.4 / 142 against 51.4 / 64.4 / 75.0 / 95.8 / 141, 1 GB 327 against 331.
// The limits have stayed where they were: which kernel a plan's calls take is pinned at them.)
constexpr uint64_t kDefaultTileBytes = 1ull << 15;
constexpr uint64_t kSmallTileBytes = 1ull << 13;
constexpr uint64_t kSmallBufferBytes = 112ull << 20;   // blocks, whatever the layout
constexpr uint64_t kMediumBufferBytes = 192ull << 20;  // blocks if fewer than half of the tiles are on lines
constexpr uint64_t kCrowdedShare = 16;  // blocks if a tile in so many holds more than four tensors
// Up to here a pass in blocks loads through the caches (unless the plan's flags say otherwise).  Three
// buffers in turn, plain against non-temporal loads: pack of 8 / 32 / 64 / 128 MB 11.8 / 17.4 / 27.8 / 60.1
// against 12.1 / 20.9 / 35.7 / 58.5 us, restore 12.2 / 18.8 / 29.9 / 61.0 against 13.6 / 20.5 / 35.5 / 59.3.
constexpr uint64_t kWarmBytes = 96ull << 20;
// Above, a restore in blocks, which is then one of small tensors, goes through the caches both ways: the L2 puts the lines
// together that two tensors, or two rows of one that lies off the lines, share.  Below, the first pass over a received buffer,
// often the only one, loses more by it than a repeated one gains.  Both non-temporal / both plain, medians of first passes over new
// states and of repeated ones, us, tensors of 5 KiB, 0.45 / 0.6 / 0.8 / 0.9 GB 196 / 252 / 333 / 373 and 176 / 235 / 312 / 350 against
// 218 / 274 / 349 / 389 and 178 / 236 / 310 / 348 (the first passes with long runs and non-temporal 214 / 268 / 347 / 389), 0.95 / 1 / 1.1 GB
// 397 / 423 / 462 and 370 / 400 / 422 against 403 / 430 / 460 and 366 / 395 / 423, 1.4 / 2 / 4 GB 582 / 823 / 1643 and 549 / 777 / 1540 against
// 577 / 806 / 1605 and 544 / 768 / 1510, of 2 KB, 1 / 2 GB 447 / 883 and 437 / 870 against 456 / 882 and 443 / 877, of 1 KB, 0.6 GB 310
// and 276 against 312 and 280.
constexpr uint64_t kCachedRestoreBytes = 896ull << 20;
constexpr uint64_t kListBytes = 256ull << 20;  // listed chunks of one launch go in blocks up to here
constexpr uint64_t kVerifyTileBytes = 1ull << 16;

}  // namespace ffsnap
