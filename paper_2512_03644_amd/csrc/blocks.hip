// Pack, restore and verify in blocks of 8 KiB: the path of small buffers and of lists of small
// tensors (launch_tiles in kernels.hip has the rule).
//
// One wavefront takes one block: 8 rows of 1 KiB, lane l of a row its 16 bytes ("slot") at 16 l.  All
// 8 loads are up front, the block's CRC register comes from the matrix cores (matrix_fold.h: a dword of
// every lane at a time, weights in LDS), and the wavefronts of a workgroup that are at the same chunk
// sum their registers in LDS before one of them delivers the sum with an atomic.  A block is a
// quarter of a default tile and its chain of dependent steps is short: the weights are fetched beside
// the data, and the lane's constant covers the place in the run.  That is what a launch of a few
// thousand wavefronts or less is made of.
//
// What bounds a small call is that chain and the launch itself.  With Horner steps through byte tables in
// place of the matrix product, 124 lookups a lane and block, the wavefronts of a compute unit queued at its
// LDS, all at the same time: pack of 32 MB 18.9 us and 14.5 with the product, restore 18.9 and 14.8, verify of 41 / 3.2 MB
// 16.6 / 9.6 and 11.5 / 6.1.  With the chain's ends shorter (block_behind_args, few_tensors, kAhead) 12.9, 13.4 and 10.7 / 5.5.  A
// copy of so many bytes in this shape, with these loads, stores and order, takes 12.3 for 32 MB (three sets in turn, as those;
// one set 10.8, where a pack takes 11.4 and a restore 11.9) and 4.6 for 3 MB, which pack and restore do in 7.1 / 7.4: what a call
// of a few MB spends behind and in front of its rows hides behind other wavefronts' rows in one of 32.
// On 1 GB of 5 KiB tensors, where the lookups hid behind the memory, a restore took 407 us, 396 with the product, and on
// another machine 431 so and 395 now (kShortXcdGroup, kCachedRestoreBytes), though the weights leave room for two workgroups on a compute unit and
// the tables left it for three; a long pack takes half the weights, and has three (block_kernel_lean).
//
// A call is one launch where it can be (T.tally set): the sums of a chunk meet in a 64-bit word of the
// plan's tally, which starts at zero, and whoever completes the word writes the chunk's result and
// sets the word back to zero.  Otherwise -- a call on another stream than the default one, or under
// capture -- the sums are XORed into the caller's own array between a preset and a finishing kernel.
//
// A block that lies inside one tensor needs one address, one of up to four tensors (few_tensors) a comparison with
// each boundary.  In any other the wavefront first puts the block's tensors into a table in LDS (base address and end of each); every tensor marks the first
// slot that starts in it, and a running maximum over the slots gives every lane its tensor: no
// search.  Slots that straddle a boundary are listed and moved by groups of eight lanes, a halfword
// each, all of the block's at once.  The cost is the same for 2 or 100 tensors in a block; with the
// tile kernel's row-by-row path a block of small tensors was 32 dependent chains in a row.
#include "kernels.hpp"

#include "fold.h"
#include "hold.h"
#include "matrix_fold.h"
#include "tally.h"

namespace ffsnap {

namespace {

constexpr int kRows = kBlockBytes / 1024;
constexpr int kWaves = 8, kWavesLog2 = 3;
static_assert(kWaves == 1 << kWavesLog2);
constexpr int kThreads = kWaves * kWaveSize;
constexpr int kSlots = kBlockBytes / 16;
constexpr uint32_t kMaxSegs = 128;  // tensors of a block that the table holds
constexpr int kPieces = 4;          // tensors of a block that need no table
static_assert(kMaxSegs <= 256, "a place in the table is 8 bits");

typedef uint16_t u16_alias __attribute__((may_alias));
typedef u32x4 u32x4_alias __attribute__((may_alias));

// LEAN: the weights of the last four rows alone.  The first four are taken on their own with the same, as a register
// that lies four rows further from the end; 110 instructions more for a block, but room for a third workgroup
// on a compute unit beside the scratch of blocks of several tensors.
template <bool LEAN>
struct BlockLds {
    static constexpr int kFirstRow = LEAN ? kRows / 2 : 0;
    u32x4 weight[(kRows - kFirstRow) * 4][kWaveSize];  // of every dword of a lane's slots, from that row on
    uint64_t sum[kWaves];      // per run (at its first wavefront's place): its registers, and who has added them
    uint32_t verdict[kWaves];  // on the run's chunk, of a restore that waits for it: 0 none yet, 2 sound, 3 damaged
};

// A wavefront's own scratch for a block of several tensors.
struct GatherLds {
    u32x4 seg[kMaxSegs];  // x, y: address of the block's byte 0 if it were in that tensor; z: end of
                          // the tensor relative to the block, at most kBlockBytes
    union {
        uint32_t mark[kSlots];          // highest tensor that has started at or before the slot
        u32x4_alias fix[kMaxSegs + 1];  // later: contents of the straddling slots
    };
    uint32_t list[kMaxSegs + 1];        // straddling slots: tensor of their first byte << 16 | slot
};

__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// inclusive running maximum over the lanes
__device__ __forceinline__ uint32_t scan_max(uint32_t v)
{
    auto step = [&](uint32_t o) { v = o > v ? o : v; };
    step(__builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false));  // row_shr:1
    step(__builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false));  // row_shr:2
    step(__builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false));  // row_shr:4
    step(__builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false));  // row_shr:8
    step(__builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false));  // row_bcast:15 into rows 1, 3
    step(__builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false));  // row_bcast:31 into rows 2, 3
    return v;
}

__device__ __forceinline__ uint32_t lanes_below(uint64_t mask)
{
    return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0));
}

// Where a lane's slots of the block's rows lie on the tensor side.
struct Place {
    uint32_t seg[kRows / 4];   // place in GatherLds::seg of the tensor of the slot's first byte, 8 bits a row
    uint64_t straddle[kRows];  // (wave-uniform) lanes whose slot lies in several tensors or holds the end
    uint64_t plain[kRows];     // (wave-uniform) lanes whose slot lies in one tensor
    uint32_t n_list;           // straddling slots
};

// The plan's entry of the k-th of n tensors from `first` on (of the last, if there are fewer).
struct Tensor {
    uint64_t begin, end, at;
};
__device__ __forceinline__ Tensor tensor_entry(const TileTables& T, const uint32_t first, const uint32_t n, uint32_t k)
{
    k = k < n ? k : n - 1;
    return Tensor{T.seg_off[first + k], T.seg_off[first + k + 1], T.seg_ptr[first + k]};
}

// The block that starts at stream offset s is touched by no tensors but the n from `first` on, which
// holds s; `end` of the block's bytes are payload.  mine: the entry of the lane-th of them.
__device__ __forceinline__ void locate(const TileTables& T, GatherLds& G, const uint32_t first,
                                       const uint32_t n, const uint64_t s, const uint32_t end,
                                       const int lane, const Tensor& mine, Place& P)
{
    u32x4_alias* const m4 = reinterpret_cast<u32x4_alias*>(G.mark);
    static_assert(kSlots == 8 * kWaveSize, "two 16-byte stores per lane clear the marks");
    m4[lane] = u32x4{0, 0, 0, 0};
    m4[lane + kWaveSize] = u32x4{0, 0, 0, 0};
    wave_sync();
    for (uint32_t k = lane; k < n; k += kWaveSize) {
        const Tensor t = k < kWaveSize ? mine : tensor_entry(T, first, n, k);
        const uint64_t base = t.at + (s - t.begin);
        const uint32_t stop = t.end - s < uint64_t(kBlockBytes) ? static_cast<uint32_t>(t.end - s) : kBlockBytes;
        G.seg[k] = u32x4{static_cast<uint32_t>(base), static_cast<uint32_t>(base >> 32), stop, 0};
        if (k) {
            const uint64_t slot = (t.begin - s + 15) / 16;  // first slot that starts in this tensor
            if (slot < kSlots) atomicMax(&G.mark[slot], k);
        }
    }
    wave_sync();
    uint32_t mark[kRows];
    static_for<kRows>([&](auto r) { mark[r] = G.mark[r * kWaveSize + lane]; });
    uint32_t seen = 0, n_list = 0;
    static_for<kRows>([&](auto r) {
        const uint32_t up = scan_max(mark[r]);
        const uint32_t j = up > seen ? up : seen;
        seen = __builtin_amdgcn_readlane(j, 63);
        const u32x4 e = G.seg[j];
        const uint32_t rel = r * 1024 + 16 * lane;
        P.seg[r / 4] = r % 4 ? P.seg[r / 4] | j << (8 * (r % 4)) : j;
        const bool in = rel < end;
        const bool one = in && rel + 16 <= e.z;
        P.plain[r] = __ballot(one);
        P.straddle[r] = __ballot(in && !one);
        if (in && !one) G.list[n_list + lanes_below(P.straddle[r])] = j << 16 | (r * kWaveSize + lane);
        n_list += __builtin_popcountll(P.straddle[r]);
    });
    P.n_list = n_list;
    wave_sync();
}

// The straddling slots, eight lanes each: move(address of the halfword, its place in G.fix).
template <class Fn>
__device__ __forceinline__ void each_straddling_half(GatherLds& G, const Place& P, const uint32_t n,
                                                     const uint32_t end, const int lane, Fn&& move)
{
    for (uint32_t i = lane; i < 8 * P.n_list; i += kWaveSize) {
        const uint32_t entry = G.list[i >> 3];
        uint32_t j = entry >> 16;
        const uint32_t pos = (entry & 0xFFFFu) * 16 + 2 * (i & 7);
        if (pos >= end) {
            move(uint64_t(0), i);
            continue;
        }
        u32x4 e = G.seg[j];
        while (pos >= e.z && j + 1 < n) e = G.seg[++j];
        move((uint64_t(e.y) << 32 | e.x) + pos, i);
    }
}

// More tensors than the table holds (less than 64 bytes each): every lane walks through its slots
// halfword by halfword from a bisection of its own.
template <bool PACK>
__device__ __noinline__ u32x4 move_crowded_row(const uint64_t* __restrict__ seg_off,
                                               const uint64_t* __restrict__ seg_ptr, uint32_t first,
                                               uint32_t n, uint64_t pos, uint64_t payload, u32x4 w)
{
    uint32_t lo = first, hi = first + n - 1;
    while (lo < hi) {
        const uint32_t mid = lo + (hi - lo + 1) / 2;
        if (seg_off[mid] <= pos) lo = mid; else hi = mid - 1;
    }
    uint64_t a = seg_off[lo], b = seg_off[lo + 1], base = seg_ptr[lo];
    uint32_t d[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int u = 0; u < 8; u++) {
        const uint64_t p = pos + 2u * u;
        uint32_t h = 0;
        if (p < payload) {
            while (p >= b) {
                lo++;
                a = b;
                b = seg_off[lo + 1];
                base = seg_ptr[lo];
            }
            uint16_t* const q = reinterpret_cast<uint16_t*>(base + (p - a));
            if (PACK)
                h = *as_global(q);
            else
                *as_global(q) = static_cast<uint16_t>(d[u >> 1] >> ((u & 1) * 16));
        }
        if (PACK) d[u >> 1] = (u & 1) ? d[u >> 1] | (h << 16) : h;
    }
    return u32x4{d[0], d[1], d[2], d[3]};
}

// A block of up to kPieces tensors, the payload's end included: the boundaries stand in scalar registers and every lane
// finds its tensors' addresses by comparing.  w: the rows (restore).
// A small call ends when its last boundary block does, and by way of the table in LDS that one has two more loads and a
// microsecond of LDS between its number and its rows.  By the table / so, us: pack of 3 / 32 / 60 / 100 MB 8.2 / 14.1 /
// 23.2 / 46.2 and 7.1 / 13.3 / 22.0 / 44.1, restore of 32 / 60 MB 14.3 / 23.8 and 13.7 / 23.1, 60 MB off the lines 25.5 and
// 23.4, tensors of 5 KiB, 100 MB, pack 46.6 and 44.2, 300 MB, restore 126.9 and 123.8, 1 GB 406 and 400.  Not where a block
// is held, nor in packs with half the weights: they have no registers for it (300 MB of 5 KiB 147 and 181, pack 116 and 126).
template <int MODE, int HINT, class Ready, class Fold>
__device__ __forceinline__ void few_tensors(const TileTables& T, GatherLds& G, uint8_t* bp, u32x4 (&w)[kRows],
                                            const uint32_t first, const uint64_t s, const uint32_t end,
                                            const bool folding, const int lane, Ready&& tables_ready, Fold&& fold)
{
    constexpr bool kSegNT = (HINT & 1) != 0, kBufNT = (HINT & 2) != 0;
    static_assert(kPieces == 4, "the sums below are written out");
    uint64_t a[kPieces], p[kPieces];  // where the tensors begin in the stream, and their addresses
    static_for<kPieces>([&](auto k) {
        a[k] = table_entry(T.seg_off, first + k < T.n_seg ? first + k : T.n_seg);
        p[k] = table_entry(T.seg_ptr, first + k < T.n_seg ? first + k : T.n_seg - 1);
    });
    // address of the block's byte 0 if it were in the tensor; where the next ones begin in the block (kBlockBytes: not in
    // it)
    auto base = [&](int k) { return p[k] + (s - a[k]); };
    auto bound = [&](int k) {
        return a[k] <= s ? 0u : a[k] - s < uint64_t(kBlockBytes) ? static_cast<uint32_t>(a[k] - s) : uint32_t(kBlockBytes);
    };
    const uint64_t b0 = base(0), step1 = base(1) - b0, step2 = base(2) - base(1), step3 = base(3) - base(2);
    const uint32_t c1 = bound(1), c2 = bound(2), c3 = bound(3);
    auto at = [&](uint32_t rel) {
        return reinterpret_cast<uint8_t*>(b0 + (rel >= c1 ? step1 : 0) + (rel >= c2 ? step2 : 0) + (rel >= c3 ? step3 : 0) + rel);
    };
    // the slots that hold a boundary in their middle, the last one that of the payload's end; kNone where there is none, or
    // it is in the list already (0 <= c1 <= c2 <= c3 <= end or kBlockBytes)
    constexpr uint32_t kNone = 0xFFFFFFFFu;
    auto cut = [&](uint32_t before, uint32_t c) {
        return c < kBlockBytes && (c & 15u) && before <= (c & ~15u) ? c & ~15u : kNone;
    };
    const uint32_t q0 = cut(0, c1), q1 = cut(c1, c2), q2 = cut(c2, c3), q3 = cut(c3, end);
    // lane 8 k + u has halfword u of the k-th of them
    const uint32_t q = lane < 8 ? q0 : lane < 16 ? q1 : lane < 24 ? q2 : lane < 32 ? q3 : kNone;
    const uint32_t half = q + 2u * (lane & 7);
    const bool moves = q != kNone && half < end;
    u16_alias* const fix = reinterpret_cast<u16_alias*>(G.fix);
    const uint32_t lane16 = 16u * lane;
    auto rel = [&](auto r) { return r * 1024 + lane16; };
    auto cut_row = [&](auto r) {  // (wave-uniform)
        return q0 / 1024 == uint32_t(r) || q1 / 1024 == uint32_t(r) || q2 / 1024 == uint32_t(r) || q3 / 1024 == uint32_t(r);
    };
    auto slot = [&](uint32_t x) { return x == q0 ? 0u : x == q1 ? 1u : x == q2 ? 2u : x == q3 ? 3u : kNone; };
    auto plain = [&](uint32_t x) { return x < end && x != q0 && x != q1 && x != q2 && x != q3; };
    if (MODE == kPack) {
        uint32_t h = 0;
        if (moves) h = *as_global(reinterpret_cast<const uint16_t*>(at(half)));
        static_for<kRows>([&](auto r) {
            w[r] = u32x4{0, 0, 0, 0};
            if (plain(rel(r))) w[r] = load16_unaligned<kSegNT>(at(rel(r)));
        });
        tables_ready();
        if (lane < 32) fix[lane] = static_cast<uint16_t>(h);
        wave_sync();
        static_for<kRows>([&](auto r) {
            if (cut_row(r)) {
                const uint32_t k = slot(rel(r));
                if (k != kNone) w[r] = G.fix[k];
            }
            store16_stream<kBufNT>(bp + rel(r), w[r]);
            if (!folding) return;
            __builtin_amdgcn_sched_barrier(0);
            fold(r);
            __builtin_amdgcn_sched_barrier(0);
        });
        return;
    }
    tables_ready();
    static_for<kRows>([&](auto r) {
        if (cut_row(r)) {
            const uint32_t k = slot(rel(r));
            if (k != kNone) G.fix[k] = w[r];
        }
        if (plain(rel(r))) store16_unaligned<kSegNT>(at(rel(r)), w[r]);
    });
    wave_sync();
    if (moves) *as_global(reinterpret_cast<uint16_t*>(at(half))) = fix[lane];
    if (folding) static_for<kRows>([&](auto r) { fold(r); });
}

// One block.  tables_ready() is the workgroup's barrier; every wavefront calls it exactly once, each in
// the branch it takes.  HOLD (restore): the block is folded first, and stored only if permit(), which takes
// the sums to the tally and waits for the chunk's verdict, says so.
template <int MODE, int HINT, bool HOLD, bool LEAN, class Ready, class Permit>
__device__ __forceinline__ void block_rows(const TileTables& T, BlockLds<LEAN>& lds, GatherLds* gather,
                                           uint8_t* __restrict__ chunks, const uint32_t tile,
                                           const bool folding, const int lane, Ready&& tables_ready,
                                           f32x16& acc, uint32_t& first_half, Permit&& permit)
{
    constexpr bool kSegNT = (HINT & 1) != 0, kBufNT = (HINT & 2) != 0;
    const uint64_t s = static_cast<uint64_t>(tile) * kBlockBytes;
    uint8_t* const bp = chunks + s;
    const uint32_t lane16 = 16u * lane;
    // A row's place for a lane.  Held: from a copy of lane16 as old as its use, or 64-bit offsets wait in scratch memory.
    auto lane_offset = [&](auto r) {
        uint32_t v = lane16;
        if (HOLD) asm volatile("" : "+v"(v));
        return v + 1024 * r;
    };
    u32x4 w[kRows];
    if (MODE != kPack)
        static_for<kRows>([&](auto r) { w[r] = load16_stream<kBufNT>(bp + (lane16 + 1024 * r)); });
    auto fold = [&](auto r) {
        constexpr int first = BlockLds<LEAN>::kFirstRow, row = r < first ? r : r - first;
        static_for<4>([&](auto f) { matrix_add(acc, lds.weight[4 * row + f][lane], w[r][int(f)]); });
        if constexpr (LEAN && r == first - 1) {
            first_half = matrix_halves(acc);
            acc = f32x16{};
        }
        if (LEAN) __builtin_amdgcn_sched_barrier(0);  // (the weights of one row at a time)
    };
    const uint32_t entry = tile >> T.block_log2;  // of the plan's tables
    const uint32_t sub = tile - (entry << T.block_log2);
    // Where the block lies, whichever way that is: all asked for at once.
    const uint64_t tb = MODE == kVerify ? 0 : table_entry(T.tile_base, entry);
    uint32_t first = 0, last = 0;
    if (MODE != kVerify) {
        first = table_entry(T.tile_first_seg, entry);
        // the tensor of the next entry's first byte is the last that can touch this block
        const bool more = entry + 1 < T.n_tiles >> T.block_log2;
        last = table_entry(T.tile_first_seg, more ? entry + 1 : entry);
        if (!more) last = T.n_seg - 1;
    }
    if (MODE == kVerify) {
        tables_ready();
    } else if (tb) {
        uint8_t* const tp = reinterpret_cast<uint8_t*>(tb) + sub * kBlockBytes;
        if (MODE == kPack)
            static_for<kRows>([&](auto r) { w[r] = load16_unaligned<kSegNT>(tp + (lane16 + 1024 * r)); });
        tables_ready();
        if (HOLD) {
            static_for<kRows>([&](auto r) { fold(r); });
            if (!permit()) return;
        }
        // Row by row, stored and folded as it arrives: the matrix cores are at work while later rows are on
        // their way.  (Pack / restore of 32 MB with all stores in front of the fold 15.9 / 16.5 us, so
        // 15.0 / 15.6.  In the blocks of several tensors below it is the other way round: restore of 5 KiB
        // tensors, 1 GB, 407 us with the stores in front, 417 row by row.)
        static_for<kRows>([&](auto r) {
            if (MODE == kPack)
                store16_stream<kBufNT>(bp + (lane16 + 1024 * r), w[r]);
            else
                store16_unaligned<kSegNT>(tp + lane_offset(r), w[r]);
            if (HOLD || !folding) return;
            __builtin_amdgcn_sched_barrier(0);
            fold(r);
            __builtin_amdgcn_sched_barrier(0);
        });
        return;
    } else {
        const uint32_t end = s >= T.payload ? 0u
                             : T.payload - s < uint64_t(kBlockBytes) ? static_cast<uint32_t>(T.payload - s)
                                                                     : uint32_t(kBlockBytes);
        if constexpr (!HOLD && !LEAN) {
            if (last - first < uint32_t(kPieces) && end) {
                few_tensors<MODE, HINT>(T, *gather, bp, w, first, s, end, folding, lane, tables_ready, fold);
                return;
            }
        }
        if (sub) {  // not the entry's first block: the last tensor that starts at or before it
            uint32_t hi = last;
            while (first < hi) {
                const uint32_t mid = first + (hi - first + 1) / 2;
                if (T.seg_off[mid] <= s) first = mid; else hi = mid - 1;
            }
        }
        const uint32_t n = last - first + 1;
        if (HOLD && (end == 0 || n > kMaxSegs)) {
            tables_ready();
            static_for<kRows>([&](auto r) { fold(r); });
            if (!permit()) return;
        }
        if (end == 0) {
            if (MODE == kPack) static_for<kRows>([&](auto r) { w[r] = u32x4{0, 0, 0, 0}; });
            if (!HOLD) tables_ready();
        } else if (n > kMaxSegs) {
#pragma unroll 1
            for (int r = 0; r < kRows; r++) {
                u32x4 x = {0, 0, 0, 0};
                if (MODE != kPack) static_for<kRows>([&](auto k) { if (k == r) x = w[k]; });
                x = move_crowded_row<MODE == kPack>(T.seg_off, T.seg_ptr, first, n,
                                                    s + 1024 * r + lane16, T.payload, x);
                if (MODE == kPack) static_for<kRows>([&](auto k) { if (k == r) w[k] = x; });
            }
            if (!HOLD) tables_ready();
        } else {
            GatherLds& G = *gather;
            Place P;
            // The tensors' entries are on their way beside the rows.  A wavefront of a restore passes the barrier when it
            // knows where its rows go: others, whose stores are behind it, wait for no stores of this one's.  With the
            // entries asked for one after the other behind the rows and the barrier behind the stores / so, us, restore of
            // 2 KB tensors, 40 / 200 MB, 24.2 / 94.0 and 22.4 / 90.8, of 5 KiB, 1 GB, 409 and 404, 24 listed chunks of them 48.2
            // and 45.5, 60 MB off the lines 28.5 and 25.3; pack of 2 KB tensors 19.8 / 79.3 and 19.4 / 77.7, of 5 KiB 367 and
            // 357.  (The barrier in front of locate(): 21.8 / 91.1, 406, 44.4, 24.6, but 32 MB on the lines 14.8 and 15.0.)
            const Tensor mine = tensor_entry(T, first, n, lane);
            locate(T, G, first, n, s, end, lane, mine, P);
            if (!HOLD && MODE == kRestore) tables_ready();
            if (HOLD) {
                tables_ready();
                static_for<kRows>([&](auto r) { fold(r); });
                if (!permit()) return;
            }
            auto slot_in_list = [&](int r) {  // place of this lane's straddling slot of row r
                uint32_t before = 0;
                static_for<kRows>([&](auto k) { before += k < r ? __builtin_popcountll(P.straddle[k]) : 0; });
                return before + lanes_below(P.straddle[r]);
            };
            auto bit = [&](uint64_t mask) { return ((mask >> lane) & 1) != 0; };
            // (an address per row would be 16 registers; the table is still there)
            auto addr = [&](auto r) {
                const u32x4 e = G.seg[(P.seg[r / 4] >> (8 * (r % 4))) & 255u];
                return reinterpret_cast<uint8_t*>((uint64_t(e.y) << 32 | e.x) + lane_offset(r));
            };
            if (MODE == kPack) {
                static_for<kRows>([&](auto r) {
                    w[r] = u32x4{0, 0, 0, 0};
                    if (bit(P.plain[r]))
                        w[r] = load16_unaligned<kSegNT>(addr(r));
                });
                each_straddling_half(G, P, n, end, lane, [&](uint64_t addr, uint32_t i) {
                    const uint16_t h = addr ? *as_global(reinterpret_cast<const uint16_t*>(addr)) : uint16_t(0);
                    reinterpret_cast<u16_alias*>(G.fix)[i] = h;
                });
                wave_sync();
                static_for<kRows>([&](auto r) {
                    if (bit(P.straddle[r])) w[r] = G.fix[slot_in_list(r)];
                });
            } else {
                static_for<kRows>([&](auto r) {
                    if (bit(P.straddle[r])) G.fix[slot_in_list(r)] = w[r];
                });
                wave_sync();
                static_for<kRows>([&](auto r) {
                    if (bit(P.plain[r])) store16_unaligned<kSegNT>(addr(r), w[r]);
                });
                each_straddling_half(G, P, n, end, lane, [&](uint64_t addr, uint32_t i) {
                    if (addr) *as_global(reinterpret_cast<uint16_t*>(addr)) = reinterpret_cast<const u16_alias*>(G.fix)[i];
                });
            }
            if (MODE == kPack) tables_ready();
        }
        if (MODE == kPack)
            static_for<kRows>([&](auto r) { store16_stream<kBufNT>(bp + (lane16 + 1024 * r), w[r]); });
    }
    if (!HOLD && folding) static_for<kRows>([&](auto r) { fold(r); });
}

// The tables, the buffer and, behind them, the size of the grid (or of the list).
constexpr int kBlockArgs = sizeof(TileTables) + sizeof(uint8_t*) + 4;

template <int MODE, int HINT, bool LISTED, bool HOLD = false, bool LEAN = false>
__device__ __forceinline__ void block_body(const TileTables& T, uint8_t* __restrict__ chunks,
                                           const ChunkList* list)
{
    const uint32_t block = block_behind_args<0, kBlockArgs>();
    __shared__ BlockLds<LEAN> lds;
    constexpr int kFirst = BlockLds<LEAN>::kFirstRow * 4 * kWaveSize;  // of the weights, as 16-byte words
    __shared__ GatherLds gather[MODE == kVerify ? 1 : kWaves];
    const int lane = threadIdx.x & (kWaveSize - 1);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWaveSize);
    constexpr int kEach = (kRows * 4 * kWaveSize - kFirst) / kThreads;
    u32x4 tab[kEach];
    static_for<kEach>([&](auto i) {
        tab[i] = *as_global(reinterpret_cast<const u32x4*>(T.block_tab) + kFirst + i * kThreads + threadIdx.x);
    });
    // Of the multiplication that a wavefront ends with, what does not need its data: while that is on its way.  (Behind it,
    // with a run's sum and the count of its wavefronts in two LDS words instead of one: pack / restore of 32 MB 13.3 / 13.7
    // us, now 13.0 / 13.4.  Not where registers are short: a verify has room for three workgroups on a compute unit without,
    // for two with: 100 / 180 MB 21.4 / 36.3 and 23.8 / 38.5, 3 MB 5.17 and 5.09.)
    constexpr bool kAhead = !HOLD && !LEAN && MODE != kVerify;
    uint32_t lane_c = 0, times[16];
    auto tables_ready = [&] {
        if (kAhead) gf2_multiples(times, lane_c);
        static_for<kEach>([&](auto i) { (&lds.weight[0][0])[i * kThreads + threadIdx.x] = tab[i]; });
        if (threadIdx.x < kWaves) lds.sum[threadIdx.x] = lds.verdict[threadIdx.x] = 0;
        workgroup_barrier();
    };
    const uint32_t slot = xcd_order(block, gridDim.x, T.xcd_group) * kWaves + wave;
    const uint32_t count = LISTED ? list->n << T.tpc_log2 : T.n_list ? T.n_list : T.n_tiles;
    bool active = slot < count;
    uint32_t chunk = 0, tile = 0;
    if (active) {
        if (LISTED) {
            chunk = list->id[slot >> T.tpc_log2];
            tile = (chunk << T.tpc_log2) + (slot & (T.tiles_per_chunk - 1));
        } else {
            tile = T.tile_begin + slot;
            chunk = tile >> T.tpc_log2;
        }
        if (T.skip_bad) active = !table_entry(T.skip_bad, chunk);
    }
    // the wavefronts of this workgroup that are at the same chunk
    const uint32_t run_log2 = T.tpc_log2 < uint32_t(kWavesLog2) ? T.tpc_log2 : uint32_t(kWavesLog2);
    const uint32_t run = 1u << run_log2, run_index = (tile & (T.tiles_per_chunk - 1)) >> run_log2;
    const uint32_t in_run = wave & (run - 1), lead = wave - in_run;
    const bool folding = T.acc != nullptr;
    uint32_t lane_c_first = 0, bit_at_end = 0, want = 0;
    if (folding) {
        // x^(8 * bytes between the end of the lane's slot in a row and the end of the run), and what bit
        // `lane` of the run's register is at the end of the chunk
        lane_c = T.block_tab[kRows * 4 * kWeightWords + (run - 1 - in_run) * kWaveSize + lane];
        if (LEAN) lane_c_first = T.block_tab[kRows * 4 * kWeightWords + (kWaves + run - 1 - in_run) * kWaveSize + lane];
        bit_at_end = T.run_tab[run_index * 32 + (lane & 31)];
        // (asked for by all, though the chunk's last run alone needs it: it is there by then)
        if (MODE != kPack && T.tally) want = table_entry(T.want, chunk);
    }
    f32x16 acc = {};
    uint32_t first_half = 0;
    // the block's register on its way; true in the wavefront (lane 0) that has taken the run's to the chunk
    auto deliver = [&] {
        uint32_t v = kAhead ? gf2_mul_half(matrix_halves(acc), times) : gf2_mul_half(matrix_halves(acc), lane_c);
        if (LEAN) v ^= gf2_mul_half(first_half, lane_c_first);
        v = wave_xor(v);
        if (run > 1) {
            uint32_t complete = 0;
            if (lane == 0) complete = run_complete(lds.sum[lead], in_run, run, v) ? 1u : 0u;
            if (!__builtin_amdgcn_readfirstlane(complete)) return false;
            v = __builtin_amdgcn_readfirstlane(v);
        }
        v = wave_xor(lane < 32 && ((v >> lane) & 1u) ? bit_at_end : 0u);
        if (lane != 0) return false;
        if (T.tally)
            tally_run<MODE>(T, v, chunk, run_index, T.tiles_per_chunk >> run_log2,
                            (slot >> T.tpc_log2), count >> T.tpc_log2, want);
        else
            atomicXor(T.acc + chunk, v);
        return true;
    };
    // (as in hold.h: one wavefront of the run waits for the others, and not for ever)
    auto permit = [&] {
        volatile uint32_t* const said = &lds.verdict[lead];
        uint32_t verdict = 0;
        if (__builtin_amdgcn_readfirstlane(deliver() ? 1u : 0u)) {
            verdict = await_verdict(T, chunk);
            static_assert(!HOLD || !LEAN, "all weights");
            if (!verdict)  // (the block stays in its registers meanwhile: room for two rows)
                verdict = find_verdict<2>(T.verdict + chunk, T.epoch, T.want + chunk, T.affine,
                                          (const FF_LDS u32x4*)&lds.weight[0][0],
                                          chunks + (uint64_t(chunk) << T.tpc_log2) * kBlockBytes, 1u << T.tpc_log2,
                                          T.block_tab[kRows * 4 * kWeightWords + lane], lane);
            *said = verdict;
        } else {
            while (!(verdict = __builtin_amdgcn_readfirstlane(*said))) __builtin_amdgcn_s_sleep(1);
        }
        return verdict == 2;
    };
    if (MODE != kPack && T.direct && !T.n_bad_add && slot == gridDim.x * kWaves - 1 && lane == 0)
        open_count(T.state, T.epoch, T.n_bad);
    if (active)
        block_rows<MODE, HINT, HOLD, LEAN>(T, lds, &gather[MODE == kVerify ? 0 : wave], chunks, tile, folding, lane,
                                     tables_ready, acc, first_half, permit);
    else
        tables_ready();
    if (!HOLD && active && folding) deliver();
}

// (two workgroups on a compute unit: the weights and the scratch of blocks of several tensors leave room for no more)
template <int MODE, int HINT>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4))) void block_kernel(TileTables T, uint8_t* __restrict__ chunks)
{
    block_body<MODE, HINT, false>(T, chunks, nullptr);
}

// Three of them, for packs of several rounds: two / three, us, 600-byte tensors 150 / 300 MB 69.3 / 65.5, 127.1 / 120.4 (with
// byte tables, three workgroups, 68.8, 125.3), ragged ones of 3.3 KB 123.0 / 116.7, 60 of 2.5 MB off the lines 62.4 / 60.8,
// 1 GB of 2.5 KB 374 / 372.  A restore spills for it and is 0-4 % slower.
template <int MODE, int HINT>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(6))) void block_kernel_lean(TileTables T, uint8_t* __restrict__ chunks)
{
    block_body<MODE, HINT, false, false, true>(T, chunks, nullptr);
}

// Restore of what verifies, in one pass: every wavefront holds its block until its chunk's verdict is there.
template <int HINT>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4))) void block_kernel_held(
    TileTables T, uint8_t* __restrict__ chunks)
{
    block_body<kRestore, HINT, false, true>(T, chunks, nullptr);
}

// The blocks of the chunks in `list`, which travels in the kernel arguments, instead of a range.
template <int MODE, int HINT>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4))) void block_kernel_listed(
    TileTables T, uint8_t* __restrict__ chunks, ChunkList list)
{
    block_body<MODE, HINT, true>(T, chunks, &list);
}

template <int MODE>
void launch(const TileTables& t, uint8_t* chunks, unsigned grid, hipStream_t stream)
{
#define FF_BLOCKS(H) \
    hipLaunchKernelGGL((block_kernel<MODE, H>), dim3(grid), dim3(kThreads), 0, stream, t, chunks)
    switch (t.hint & 3) {
    case 0: FF_BLOCKS(0); break;
    case 1: FF_BLOCKS(1); break;
    case 2: FF_BLOCKS(2); break;
    default: FF_BLOCKS(3); break;
    }
#undef FF_BLOCKS
}

}  // namespace

void build_run_tab(uint32_t* tab, uint64_t runs, uint64_t run_bytes)
{
    uint32_t end = kX32;
    const uint32_t x_run = gf2_xpow(8 * run_bytes);
    for (uint64_t k = runs; k-- > 0; end = gf2_mul(end, x_run)) {
        uint32_t v = end;
        for (int i = 31; i >= 0; i--, v = gf2_mulx(v)) tab[32 * k + i] = v;
    }
}

void build_block_tab(uint32_t* tab)
{
    // a dword enters times x^(8 * bytes from its end to the end of the last row's slot of lane 31 or 63)
    for (int r = 0; r < kRows; r++)
        for (int f = 0; f < 4; f++) {
            const uint32_t high = gf2_xpow(8ull * 1024 * (kRows - 1 - r) + 32 * (3 - f));
            build_matrix_weights(tab + (4 * r + f) * kWeightWords, gf2_mul(high, gf2_xpow(8 * 512)), high);
        }
    const uint32_t x_block = gf2_xpow(8ull * kBlockBytes);
    uint32_t* const lanes = tab + 4 * kRows * kWeightWords;
    for (int lane = 0; lane < kWaveSize; lane++) {
        uint32_t v = matrix_lane_factor(lane, 8 * 16);
        const uint32_t x_half = gf2_xpow(4ull * kBlockBytes);
        for (int k = 0; k < kWaves; k++, v = gf2_mul(v, x_block)) {
            lanes[k * kWaveSize + lane] = v;
            lanes[(kWaves + k) * kWaveSize + lane] = gf2_mul(v, x_half);
        }
    }
}

// Workgroups for `count` blocks; with T.direct one more, whose last wavefront has nothing else to do than to open
// the count.
static unsigned grid_of(const TileTables& t, TileMode mode, uint64_t count)
{
    return static_cast<unsigned>((count + kWaves - 1) / kWaves) + (mode != kPack && t.direct && !t.n_bad_add ? 1u : 0u);
}

hipError_t launch_held(const TileTables& t, void* chunks, hipStream_t stream)
{
    if (!t.tally || !t.verdict || !t.acc || t.n_list || t.tile_begin) return hipErrorInvalidValue;
    uint8_t* const c = static_cast<uint8_t*>(chunks);
    if (tiles_are_blocks(t)) {
        const unsigned grid = grid_of(t, kRestore, t.n_tiles);
        const auto kernel = t.hint == kHintWarm(kRestore) ? block_kernel_held<kHintWarm(kRestore)> : block_kernel_held<3>;
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(kThreads), 0, stream, t, c);
    } else if (t.tile_rows == hold::kRows) {
        const unsigned grid = (t.n_tiles + hold::kWaves - 1) / hold::kWaves;
        hipLaunchKernelGGL(hold::tile_kernel_held<3>, dim3(grid), dim3(hold::kThreads), 0, stream, t.seg_off, t.seg_ptr,
                           t.tile_first_seg, t.tile_base, t.tile_shift, t, c);
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_blocks(TileMode mode, const TileTables& t, void* chunks, hipStream_t stream,
                         const ChunkList* list)
{
    uint8_t* c = static_cast<uint8_t*>(chunks);
    const uint64_t count = list ? uint64_t(list->n) << t.tpc_log2 : t.n_list ? t.n_list : t.n_tiles;
    if (count == 0) return hipSuccess;
    if (t.tile_rows != kRows || (list && (list->n > kMaxListedChunks || mode == kPack)) || count > 0x7FFFFFF0ull)
        return hipErrorInvalidValue;
    const unsigned grid = grid_of(t, mode, count);
    if (list) {
        const auto restore = t.hint == kHintWarm(kRestore) ? block_kernel_listed<kRestore, kHintWarm(kRestore)>
                                                           : block_kernel_listed<kRestore, 3>;
        const auto verify = t.hint == kHintWarm(kVerify) ? block_kernel_listed<kVerify, kHintWarm(kVerify)>
                                                         : block_kernel_listed<kVerify, 3>;
        hipLaunchKernelGGL(mode == kRestore ? restore : verify, dim3(grid), dim3(kThreads), 0, stream, t, c, *list);
    } else {
        if (mode == kPack && count > kLeanBlocks && t.hint == 3) {
            hipLaunchKernelGGL((block_kernel_lean<kPack, 3>), dim3(grid), dim3(kThreads), 0, stream, t, c);
            return hipGetLastError();
        }
        switch (mode) {
        case kPack: launch<kPack>(t, c, grid, stream); break;
        case kRestore: launch<kRestore>(t, c, grid, stream); break;
        case kVerify: launch<kVerify>(t, c, grid, stream); break;
        }
    }
    return hipGetLastError();
}

}  // namespace ffsnap
