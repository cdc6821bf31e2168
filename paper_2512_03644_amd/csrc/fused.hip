// Fused optimizer step + snapshot for gfx950.
//
// Work tiles (layout.hpp) are blocks of up to kParamTileElems elements of one parameter group, or of
// up to kRawTileBytes bytes of a RAW segment.  One wavefront takes one sub-block: 2 rows of 256
// elements, lane l of a row taking 4 consecutive elements: 8 bytes of 16-bit gradient and 3 x 16
// bytes of fp32 master/m/v come in, the AdamW update runs in registers, and the four results go out
// twice -- in place, and at their stream offsets in the chunk buffer -- and, from the same registers,
// into the CRC of their stream, so the snapshot is never read back from memory.  Rows are aligned
// to the tensors' elements; elements of a row that are not the tile's count as zeros.
//
// A sub-block is straight-line code with all its loads up front; the registers of its four streams come
// from the matrix cores (matrix_fold.h, weights in LDS) as eight bits of each in every lane, which are
// multiplied by the lane's factors before the lanes share the streams out among themselves.
// The sub-blocks of a tile that share a workgroup sum their registers in LDS; the last one to arrive
// multiplies the sums by x^(8 * distance to the end of the chunk) and XORs them into crcs[chunk] with
// an atomic; XOR is commutative, so the result does not depend on the order in which tiles finish.  A
// prepare kernel sets crcs[] to the preset/complement term and writes the zero tail of the last chunk; a short
// step on the default stream does without it: its contributions meet in the plan's tally (add_to_tally), and
// workgroups of its own clear the tail.
//
// What bounds it: the memory system's handling of 4 load and 8 (chained: 5) store streams at once, and how
// well it does depends on where the tensors lie: one 7B shard in place takes 5.5 or 6.5 ms from one
// allocation to the next, with this kernel and any other tried.  Results are stored from registers, stream by
// stream, by two workgroups on a compute unit (three where they hold the launch at once).  Where most
// elements have an fp32 stream off its 128-byte lines, longer runs on the lines are worth a detour: the new
// master, m and v of a workgroup are laid out in LDS, and every wavefront stores 12 KiB of consecutive
// rows.  (The image used by every launch is what the second column has: 3-6 % faster on aligned lists of 60-250
// million elements in the worse placements, but 5-12 % slower from 400 million on or in the better
// placements, 10 % slower in the first passes after a pause, 10-20 % on small launches.)  One process, same
// tensors, ms: rows handed through LDS by workgroups of 8 / image for all / as now
//   7B shard, 842 million elements, aligned: a worse placement   6.60 / 6.53 / 6.50   a better one 5.65 / 6.15 / 5.47
//     the first pass after 0.3 s without work                    6.70 / 7.30 / 6.65                6.15 / 7.15 / 6.12
//   128 parameters of 4 million, aligned: worse, better          4.19 / 4.16 / 4.28                3.62 / 3.90 / 3.55
//   64 parameters of 4 million, aligned                          2.04 / 2.03 / 2.10                1.99 / 1.95 / 1.89
//   64 parameters of 4194381, off the lines                      2.57 / 2.17 / 2.07
//   30 odd-sized parameters, 354 million                         3.31 / 2.74 / 2.70
//   2000 ragged groups in fp16, 190 MB                           1.25 / 1.07 / 1.03
//   64 parameters, 2.1 million                                   0.032 / 0.026 / 0.023
// Chained: 7B 4.60 / 4.53 / 4.53, odd-sized 2.15 / 2.02 / 2.02, 64 parameters 0.031 / 0.023 / 0.023.
// With the registers from the matrix cores (all of the above had 108 lookups a lane and sub-block in byte
// tables, 64 random LDS addresses each), us: 35 fp16 parameters of 19,000 elements and 300 RAW tensors 27.7 ->
// 24.5, 96 ragged ones 34.8 -> 31.9, 2000 ragged groups 1016 -> 988, chained 20 million elements 53.1 -> 52.0;
// 64 parameters, 2.1 million, and the 7B shard the same within 0.5 %.
// Short steps since, in a kernel of their own (fused_kernel_warm), before / now, us, three sets in turn: 0.2 million elements
// 8.7 / 8.3, 2.1 million 25.2 / 21.2, chained 22.4 / 18.4, 3.2 million 33.3 / 30.7, chained 4.3 million 32.5 / 26.5.  In fp16, one
// set, 0.2 / 2.1 / 5 million 10.0 / 9.4, 22.6 / 19.7, 51.0 / 43.7, chained 10.0 / 9.4, 22.2 / 17.5, 38.4 / 31.1 (with two registers
// in scratch memory 0.1 / 1 / 2.1 million 9.50 / 13.51 / 19.7 against 9.44 / 13.33 / 19.7, chained 9.70 / 13.04 / 17.8 against 9.55 /
// 13.00 / 17.5).
#include "fused.hpp"

#include <hip/hip_fp16.h>
#include <stddef.h>

#include "fold.h"
#include "matrix_fold.h"
#include "tally.h"

namespace ffsnap {

namespace {

constexpr int kWavesPerBlock = kWavesPerGroup;
constexpr int kThreads = kWavesPerBlock * kWaveSize;
constexpr int kRowElems = 256;
constexpr int kRows = kSubElems / kRowElems;   // rows of a parameter sub-block
constexpr int kRawRows = kSubRawBytes / 1024;  // rows of a RAW sub-block
static_assert(kRows == 2 && kRawRows == 8, "sub-blocks");

__device__ __forceinline__ float bits_to_f32(uint32_t u) { return __uint_as_float(u); }
__device__ __forceinline__ uint32_t f32_to_bits(float f) { return __float_as_uint(f); }

// Two fp32 -> two bf16, the first in the low half: round to nearest even in one instruction.
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t f32_to_bf16_pair(float lo, float hi)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}

// Two fp32 -> two fp16: the hardware conversion rounds to nearest even, overflows to infinity and
// produces subnormals.
__device__ __forceinline__ uint32_t f32_to_f16_pair(float lo, float hi)
{
    return __half_as_ushort(__float2half_rn(lo)) | (uint32_t(__half_as_ushort(__float2half_rn(hi))) << 16);
}

// IEEE 754 leaves sign and payload of a NaN that an operation produces open, and processors differ
// in them.  A snapshot is compared byte for byte and CRC'd across machines, so a NaN result of the
// update is stored in one form: quiet, positive, empty payload; the 16-bit weight is rounded from
// that form, which both conversions turn into the 16-bit format's own.
constexpr uint32_t kCanonicalNaN = 0x7FC00000u;
__device__ __forceinline__ float canonical_nan(float x) { return (x != x) ? bits_to_f32(kCanonicalNaN) : x; }

// One element of the update; every operation is a separately rounded fp32 operation (the file
// is compiled with -ffp-contract=off, division and square root are correctly rounded).
// F16: the gradient is fp16 of a loss scaled by S and is multiplied by inv_scale = 1/S first.
// Otherwise it is bf16 and nothing is scaled.  BC2: the second bias correction has not yet rounded
// to one (x / 1.0f is x exactly, so the division is left out then; beta2 = 0.95 gets there at step
// 333).  A NaN in the new m or v makes the new master NaN too, so that one comparison per element
// finds the rare row whose NaNs have to be put into their stored form.
template <bool F16, bool BC2>
__device__ __forceinline__ void adam_element(const FusedConsts& C, uint32_t g_bits, float& p,
                                             float& m, float& v)
{
    const AdamConsts& k = C.adam;
    float g;
    if constexpr (F16)
        g = __half2float(__ushort_as_half(static_cast<unsigned short>(g_bits))) * C.inv_scale;
    else
        g = bits_to_f32(g_bits << 16);
    const float pd = p * k.decay;
    m = (k.b1 * m) + (k.omb1 * g);
    v = (k.b2 * v) + ((k.omb2 * g) * g);
    const float r = sqrtf(v);
    const float d = (BC2 ? r / k.bc2s : r) + k.eps;
    p = pd - (k.step_size * (m / d));
}

// fp16 infinity or NaN
__device__ __forceinline__ bool f16_nonfinite(uint32_t bits) { return (bits & 0x7C00u) == 0x7C00u; }

// the image's bytes seen as halfwords, dwords and 16-byte slots
typedef uint16_t u16_alias __attribute__((may_alias));
typedef uint32_t u32_alias __attribute__((may_alias));
typedef u32x4 u32x4_alias __attribute__((may_alias));

struct Lds {
    uint32_t sum[kWavesPerBlock][4];  // per run (at its first wavefront's place): XOR of its registers
    uint32_t arrived[kWavesPerBlock]; // wavefronts of the run that have added theirs
    uint64_t raw_sum[kWavesPerBlock]; // per run of RAW sub-blocks (run_complete)
    u32x4 wide[kRows * 4][2][kWaveSize];  // weights of the dwords of two rows of 16-byte slots
    u32x4 half[kRows * 2][2][kWaveSize];  // ... of 8-byte slots
};

// The in-place step's image: the new master, m and v of the workgroup's sub-blocks as they lie in
// their streams; behind them room for the last dword that a shifted read touches.  Dynamic LDS, so that
// only the launches that use it pay for it.
constexpr int kImgF = kWavesPerBlock * kSubElems * 4;  // bytes of one fp32 stream of a workgroup
constexpr int kImgBytes = 3 * kImgF + 16;

// Workgroups of an in-place step on a compute unit: three if they hold the launch at once, else two, made so
// by LDS that nobody uses.  Stored from registers, three against two, us: 30 parameters of 100,000 elements
// (750 workgroups) 30.9 / 32.6, 40 of 340,000 (3320) 116.4 / 114.4, 30 odd-sized ones (86,000) 3003 / 2921; 7B
// (205,000) 6640-6700 / 6470-6560 in worse placements, 5520-5540 / 5470-5480 in better ones.  Through the image 7B
// 6650-6690 / 6400-6490, 5560 / 5550, odd-sized 2890 / 2700.
constexpr unsigned kComputeUnits = 256, kSpareLds = 30 * 1024;
constexpr size_t kLds = 160 * 1024;
static_assert(3 * sizeof(Lds) <= kLds && 3 * (sizeof(Lds) + kSpareLds) > kLds && 2 * (sizeof(Lds) + kSpareLds) <= kLds,
              "two or three");
static_assert(2 * (sizeof(Lds) + kImgBytes) <= kLds && 3 * (sizeof(Lds) + kImgBytes) > kLds, "two");

// Tile registers come out of the folds without the factor x^32 that a CRC register carries.
constexpr uint32_t kX16 = gf2_xpow(16);

// A contribution to its chunk's checksum, by a lane: whoever completes the chunk writes it.
__device__ __forceinline__ void add_to_tally(const FusedConsts& C, const StepTicket k, uint32_t* __restrict__ crcs,
                                             const uint32_t chunk, uint32_t v)
{
    uint64_t now = tally_xor(C.tally + k.leaf, 1u << (k.bits & 31u), v);
    if ((now >> 32) != k.leaf_full) return;
    tally_reset(C.tally + k.leaf);
    const uint32_t leaves = (k.bits >> 8) & 63u;
    if (leaves > 1) {
        now = tally_xor(C.tally + k.root, 1u << ((k.bits >> 16) & 31u), static_cast<uint32_t>(now));
        if ((now >> 32) != (leaves == 32 ? 0xFFFFFFFFu : (1u << leaves) - 1)) return;
        tally_reset(C.tally + k.root);
    }
    crcs[chunk] = static_cast<uint32_t>(now) ^ C.affine;
}

// The ticket of stream x of the run that begins at a wavefront entry (wave-uniform).  By scalar loads, whatever the
// compiler can tell about the pointer: a vector load would wait for every store in front of it.
__device__ __forceinline__ StepTicket run_ticket(const FusedConsts& C, const uint32_t run_entry, const int x)
{
    const auto* const t = (const __attribute__((address_space(4))) u32x4*)(C.runs + 4 * run_entry);
    u32x4 k = t[0];
    static_for<3>([&](auto i) {
        const u32x4 other = t[i + 1];
        static_for<4>([&](auto j) { k[int(j)] = x == i + 1 ? other[int(j)] : k[int(j)]; });
    });
    return StepTicket{k.x, k.y, k.z, k.w};
}

// Head piece: the first two bytes of a split element, which are the last two bytes of their
// chunk.  In the low half of a dword they read M(x) * x^16, and their register is M(x) * x^32.
__device__ __forceinline__ void add_head_piece(const FusedConsts& C, uint32_t* __restrict__ crcs, const WorkTile& t,
                                               const uint32_t tile, int piece, uint32_t low_half)
{
    const uint32_t v = gf2_mul_const<kX16>(low_half);
    if (C.tally)
        add_to_tally(C, C.heads[3 * tile + piece - 4], crcs, t.chunk[piece], v);
    else
        atomicXor(&crcs[t.chunk[piece]], v);
}

// The weights on their way to LDS, first thing.  tables_ready() is a barrier of the workgroup, behind a
// wavefront's own loads (whose completion includes that of its part of the weights); every wavefront calls it
// exactly once, whether at a parameter, a RAW tile or none.  (In front of the folds instead, behind the
// stores, it costs 3 % on 50 million elements chained and 4 % on 64 small parameters.)
__device__ __forceinline__ void fetch_tables(const uint32_t* __restrict__ tabs, Lds& lds, const int wave, const int lane)
{
    static_assert(4 * kFusedWeightWords == sizeof(lds.wide) + sizeof(lds.half), "all weights");
    static_assert(offsetof(Lds, half) == offsetof(Lds, wide) + sizeof(lds.wide), "one behind the other");
    table_to_lds<kThreads, 4 * kFusedWeightWords>(tabs, &lds.wide[0][0][0], wave, lane);
    if (threadIdx.x < kWavesPerBlock * 4) (&lds.sum[0][0])[threadIdx.x] = 0;
    if (threadIdx.x < kWavesPerBlock) lds.raw_sum[threadIdx.x] = lds.arrived[threadIdx.x] = 0;
    __builtin_amdgcn_sched_barrier(0);
}
__device__ __forceinline__ void tables_ready()
{
    wait_loads<0>();
    workgroup_barrier();
    __builtin_amdgcn_sched_barrier(0);
}

// Sum of the registers of a parameter tile's run; in the run's last wavefront, on to memory.  v: the lanes
// of row j (of 16) hold the register of stream j.
__device__ __forceinline__ void deliver(const FusedConsts& C, Lds& lds, const WorkTile& t, uint32_t info, uint32_t v,
                                        const uint32_t run_entry, uint32_t* __restrict__ crcs, int lane)
{
    const int x = lane & 3;  // from here on lane x has stream x
    static_for<3>([&](auto k) {
        const uint32_t u = __builtin_amdgcn_readlane(v, 16 * (k + 1));
        v = lane == k + 1 ? u : v;
    });
    int n = 4;
    const uint32_t run = (info >> 4) & 7u, len = (info >> 8) & 15u;
    if (len > 1) {
        // LDS operations of a wavefront complete in order: the sum is complete when the count is
        uint32_t before = 0;
        if (lane < n) atomicXor(&lds.sum[run][lane], v);
        asm volatile("" ::: "memory");
        if (lane == 0) before = atomicAdd(&lds.arrived[run], 1u);
        if (__builtin_amdgcn_readfirstlane(before) + 1 != len) return;
        if (lane < n) v = *const_cast<volatile uint32_t*>(&lds.sum[run][lane]);
    }
    uint32_t s = t.shift[0], c = t.chunk[0];
    static_for<3>([&](auto k) {
        s = (x == k + 1) ? t.shift[k + 1] : s;
        c = (x == k + 1) ? t.chunk[k + 1] : c;
    });
    v = gf2_mul(v, s);
    // all streams in one chunk (any parameter much smaller than a chunk)?
    const bool one = t.chunk[0] == t.chunk[1] && t.chunk[0] == t.chunk[2] && t.chunk[0] == t.chunk[3];
    if (one) {
        v ^= __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true);
        v ^= __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true);
        n = 1;
    }
    if (lane < n) {
        if (C.tally)
            add_to_tally(C, run_ticket(C, run_entry, x), crcs, c, v);
        else
            atomicXor(&crcs[c], v);
    }
}

// s * x^(30 - 2 i), i < 16.
__device__ __forceinline__ uint32_t spread_factor(uint32_t s, const int i)
{
    const int n = 30 - 2 * i;
    static_for<4>([&](auto k) {
        uint32_t v = s;
        static_for<(2 << k)>([&](auto) { v = gf2_mulx(v); });
        s = n & (2 << k) ? v : s;
    });
    return s;
}

// Sum of the registers of a parameter tile's run; in the run's last wavefront, on to the tally.  v: the lanes of row j (of 16)
// hold the register of stream j; f: lane i of a row has spread_factor(the stream's distance to the end of its chunk, i),
// made while the data was on its way, so that the product takes two bits of v in every lane and an XOR over the row.  (One
// lane's 32 dependent steps at the end of a short step, us: 200,000 / 2.1 million elements 8.3 / 21.7, so 8.25 / 21.3,
// chained 2.1 million 19.2 and 18.6.)
__device__ __forceinline__ void deliver_to_tally(const FusedConsts& C, Lds& lds, const WorkTile& t, uint32_t info, uint32_t v,
                                                 const uint32_t f, const uint32_t run_entry, uint32_t* __restrict__ crcs,
                                                 const int lane)
{
    const int x = lane >> 4, i = lane & 15;
    const uint32_t run = (info >> 4) & 7u, len = (info >> 8) & 15u;
    if (len > 1) {
        // LDS operations of a wavefront complete in order: the sum is complete when the count is
        uint32_t before = 0;
        if (i == 0) atomicXor(&lds.sum[run][x], v);
        asm volatile("" ::: "memory");
        if (lane == 0) before = atomicAdd(&lds.arrived[run], 1u);
        if (__builtin_amdgcn_readfirstlane(before) + 1 != len) return;
        v = *const_cast<volatile uint32_t*>(&lds.sum[run][x]);
    }
    v = row_xor((((v >> (2 * i + 1)) & 1u) ? f : 0u) ^ (((v >> (2 * i)) & 1u) ? gf2_mulx(f) : 0u));
    // all streams in one chunk (any parameter much smaller than a chunk)?
    const bool one = t.chunk[0] == t.chunk[1] && t.chunk[0] == t.chunk[2] && t.chunk[0] == t.chunk[3];
    if (one)
        v = __builtin_amdgcn_readlane(v, 0) ^ __builtin_amdgcn_readlane(v, 16) ^ __builtin_amdgcn_readlane(v, 32) ^
            __builtin_amdgcn_readlane(v, 48);
    if (lane == 0 || (i == 0 && !one)) {
        uint32_t c = t.chunk[0];
        static_for<3>([&](auto k) { c = (x == k + 1) ? t.chunk[k + 1] : c; });
        add_to_tally(C, run_ticket(C, run_entry, x), crcs, c, v);
    }
}

// ---- parameter sub-block -------------------------------------------------------------------------

struct RowIn {
    u32x2 g;
    u32x4 p, m, v;
};

// Stores the elements [lo, hi) of the image (its element 0 lies `at` elements behind the tile's
// first, perhaps before it) to every fp32 output stream: in place, and to the snapshot.  The 1 KiB
// rows of all streams form one list that is cut into equal runs, so a wavefront sweeps contiguous
// memory.  Rows lie on the destination's 128-byte lines, whatever its alignment: the image
// is read at the offset that takes.  A stream's first and last row may be partial; a lane on such an
// edge moves its bytes halfword by halfword.
__device__ __forceinline__ void store_image(const WorkTile& t, const uint8_t* img, const int at,
                                            const int lo, const int hi, uint8_t* __restrict__ chunks,
                                            const int wave, const int lane)
{
    constexpr int kOut = 6;  // output o: master, m, v in place, then in the snapshot
    auto stream_of = [](int o) { return o < 3 ? o + 1 : o - 2; };
    auto dest = [&](int o) {
        const int x = stream_of(o);
        uint8_t* const base = o < 3 ? reinterpret_cast<uint8_t*>(t.ptr[x]) : chunks + t.soff[x];
        return base + 4 * static_cast<int64_t>(at);
    };
    const int vb = 4 * lo, ve = 4 * hi;
    auto rows_of = [&](int o, int& first, int& last) {  // rows [first, last) of output o
        const int m = static_cast<int>(reinterpret_cast<uint64_t>(dest(o)) & 127u);
        first = (vb + m) >> 10;
        last = (ve + m + 1023) >> 10;
    };
    int total = 0;
    static_for<kOut>([&](auto o) {
        int a, b;
        rows_of(o, a, b);
        total += b - a;
    });
    const int per = (total + kWavesPerBlock - 1) / kWavesPerBlock;
    int skip = wave * per, left = per;  // rows of the list in front of this wavefront's run, rows of the run
#pragma unroll 1
    for (int o = 0; o < kOut; o++) {
        int first, last;
        rows_of(o, first, last);
        if (skip >= last - first) {
            skip -= last - first;
            continue;
        }
        const int begin = first + skip, end = last < begin + left ? last : begin + left;
        skip = 0;
        left -= end - begin;
        uint8_t* const d0 = dest(o);
        const int m = static_cast<int>(reinterpret_cast<uint64_t>(d0) & 127u);
        const uint8_t* const im = img + (stream_of(o) - 1) * kImgF;
        const uint32_t sh = (m & 2) * 8;
        auto read = [&](int off) -> u32x4 {  // 16 bytes at byte `off` of the stream's image
            if ((m & 15) == 0) return *reinterpret_cast<const u32x4_alias*>(im + off);
            const u32_alias* r = reinterpret_cast<const u32_alias*>(im + (off & ~3));
            uint32_t d[5];
            static_for<5>([&](auto k) { d[k] = r[k]; });
            return u32x4{__builtin_amdgcn_alignbit(d[1], d[0], sh), __builtin_amdgcn_alignbit(d[2], d[1], sh),
                         __builtin_amdgcn_alignbit(d[3], d[2], sh), __builtin_amdgcn_alignbit(d[4], d[3], sh)};
        };
        auto edge_row = [&](int R) {
            const int off = 1024 * R - m + 16 * lane;
            if (off >= vb && off + 16 <= ve) {
                store16_stream<true>(d0 + off, read(off));
            } else if (off + 16 > vb && off < ve) {
#pragma unroll
                for (int u = 0; u < 8; u++) {
                    const int b = off + 2 * u;
                    if (b >= vb && b < ve)
                        *as_global(reinterpret_cast<uint16_t*>(d0 + b)) =
                            *reinterpret_cast<const u16_alias*>(im + b);
                }
            }
        };
        int R = begin;
        if (R == first) edge_row(R++);
        const int inner = end == last ? last - 1 : end;  // rows [R, inner) are whole
        for (; R + 4 <= inner; R += 4) {
            u32x4 w[4];
            static_for<4>([&](auto k) { w[k] = read(1024 * (R + k) - m + 16 * lane); });
            static_for<4>([&](auto k) { store16_stream<true>(d0 + (1024 * (R + k) - m + 16 * lane), w[k]); });
        }
        for (; R < inner; R++) {
            const int off = 1024 * R - m + 16 * lane;
            store16_stream<true>(d0 + off, read(off));
        }
        if (R < end) edge_row(R);
        if (left == 0) break;
    }
}

// The elements [lo, hi) of the sub-block (element 0 = its first place, `at` elements behind the
// tile's first element, perhaps before it) are the tile's.  WHOLE: all kSubElems of them, and no
// split element among them.
//
// Not WHOLE: lanes whose four elements are all the tile's work as in a whole sub-block; the up to
// three elements at either end that do not fill a lane's slot are updated one per lane, by lanes 0-3
// (the slot that holds lo) and 4-7 (the slot that holds hi), and handed to the lanes that own those
// slots.  What is not the tile's counts as zero.
// WARM: of a short step (fused_kernel_warm).
template <bool F16, bool CHAINED, bool BC2, bool WHOLE, bool WARM>
__device__ __forceinline__ void param_sub_block(const WorkTile& t, const uint32_t tile, const uint32_t info,
                                                const uint32_t run_entry, const int at,
                                                const int lo, const int hi,
                                                const uint8_t* __restrict__ grad,
                                                uint8_t* __restrict__ chunks,
                                                uint32_t* __restrict__ crcs, const FusedConsts& C,
                                                Lds& lds, uint8_t* img,
                                                const uint32_t* __restrict__ lane_tab, int wave, int lane)
{
    const int sub = info & 15u;
    // x^(8 * bytes between the end of the lane's column and the end of the block), in the lane's stream
    const uint32_t lane_c0 = lane_tab[(15 - sub) * 64 + lane], lane_c = lane_tab[(16 + 15 - sub) * 64 + lane];
    // wave-uniform addresses of the sub-block's element 0 in every stream; a lane adds 32 bits
    const int64_t at64 = at;
    uint8_t* const tw = reinterpret_cast<uint8_t*>(t.ptr[0]) + 2 * at64;
    uint8_t* const sw = chunks + (static_cast<int64_t>(t.soff[0]) + 2 * at64);
    uint8_t* const tp = reinterpret_cast<uint8_t*>(t.ptr[1]) + 4 * at64;
    uint8_t* const tm = reinterpret_cast<uint8_t*>(t.ptr[2]) + 4 * at64;
    uint8_t* const tv = reinterpret_cast<uint8_t*>(t.ptr[3]) + 4 * at64;
    const uint8_t* const tg = grad + 2 * (static_cast<int64_t>(t.e0) + at64);
    // where the old master, m, v come from: their tensors, or the previous snapshot
    const uint8_t* const lp = CHAINED ? C.prev + (static_cast<int64_t>(t.soff[1]) + 4 * at64) : tp;
    const uint8_t* const lm = CHAINED ? C.prev + (static_cast<int64_t>(t.soff[2]) + 4 * at64) : tm;
    const uint8_t* const lv = CHAINED ? C.prev + (static_cast<int64_t>(t.soff[3]) + 4 * at64) : tv;
    const uint32_t lane8 = 8u * lane, lane16 = 16u * lane;

    auto mine = [&](int r) {  // all four elements of the lane's slot in row r
        const int x = r * kRowElems + 4 * lane;
        return WHOLE || (x >= lo && x + 4 <= hi);
    };
    RowIn q[kRows];
    static_for<kRows>([&](auto r) {
        if (!WHOLE) q[r] = RowIn{u32x2{0, 0}, u32x4{0, 0, 0, 0}, u32x4{0, 0, 0, 0}, u32x4{0, 0, 0, 0}};
        if (mine(r)) {
            q[r].g = load8_unaligned<!WARM>(tg + (lane8 + 2 * kRowElems * r));
            q[r].p = load16_unaligned<!WARM>(lp + (lane16 + 4 * kRowElems * r));
            q[r].m = load16_unaligned<!WARM>(lm + (lane16 + 4 * kRowElems * r));
            q[r].v = load16_unaligned<!WARM>(lv + (lane16 + 4 * kRowElems * r));
        }
    });
    // edge elements: lane 0..3 element lane of the slot that holds lo, 4..7 of the slot that holds hi
    const int edge_lo = lo & ~3, edge_hi = hi & ~3;  // first elements of those slots
    const bool lo_cut = (lo & 3) || edge_lo + 4 > hi, hi_cut = (hi & 3) && edge_hi > edge_lo;
    bool has_edge = false;
    uint32_t ej = 0;  // the lane's edge element, if it has one
    uint32_t eg = 0;
    float ep = 0.f, em = 0.f, ev = 0.f;
    if (!WHOLE) {
        const int x = (lane < 4 ? edge_lo : edge_hi) + (lane & 3);
        has_edge = lane < 8 && (lane < 4 ? lo_cut : hi_cut) && x >= lo && x < hi;
        auto f32_at = [](const uint8_t* p) {  // stream offsets of fp32 segments may be 2 mod 4
            return bits_to_f32(*as_global(reinterpret_cast<const u32_a2*>(p)));
        };
        if (has_edge) {
            ej = static_cast<uint32_t>(x);
            eg = *as_global(reinterpret_cast<const uint16_t*>(tg + 2 * ej));
            ep = f32_at(lp + 4 * ej);
            em = f32_at(lm + 4 * ej);
            ev = f32_at(lv + 4 * ej);
        }
    }
    uint32_t f = 0;  // deliver_to_tally
    if constexpr (WARM) {
        if (C.tally) {
            uint32_t shift = t.shift[0];
            static_for<3>([&](auto k) { shift = (lane >> 4) == k + 1 ? t.shift[k + 1] : shift; });
            f = spread_factor(shift, lane & 15);
        }
    }
    // (Waiting for the weights alone, vmcnt counted, and for the data row by row costs 0.7 % on the 7B shard.)
    tables_ready();

    uint32_t nonfinite = 0;  // this lane's count of infinite or NaN gradient elements (fp16 only)
    uint32_t edge_w = 0, edge_nonfinite = 0;  // (of the whole wavefront)
    if (!WHOLE) {
        uint32_t wb = 0;
        // (a scalar register: a short step has no other left, and the count went to scratch memory and back)
        if (F16 && WARM) edge_nonfinite = __popcll(__ballot(f16_nonfinite(eg)));
        if (has_edge) {
            if constexpr (F16 && !WARM) nonfinite += f16_nonfinite(eg) ? 1u : 0u;
            adam_element<F16, BC2>(C, eg, ep, em, ev);
            ep = canonical_nan(ep);
            em = canonical_nan(em);
            ev = canonical_nan(ev);
            wb = (F16 ? f32_to_f16_pair(ep, 0.f) : f32_to_bf16_pair(ep, 0.f)) & 0xFFFFu;
        }
        edge_w = wb;
    }

    static_for<kRows>([&](auto r) {
        const RowIn& cur = q[r];
        const uint32_t gb[4] = {cur.g.x & 0xFFFFu, cur.g.x >> 16, cur.g.y & 0xFFFFu, cur.g.y >> 16};
        float p[4] = {bits_to_f32(cur.p.x), bits_to_f32(cur.p.y), bits_to_f32(cur.p.z), bits_to_f32(cur.p.w)};
        float m[4] = {bits_to_f32(cur.m.x), bits_to_f32(cur.m.y), bits_to_f32(cur.m.z), bits_to_f32(cur.m.w)};
        float v[4] = {bits_to_f32(cur.v.x), bits_to_f32(cur.v.y), bits_to_f32(cur.v.z), bits_to_f32(cur.v.w)};
#pragma unroll
        for (int s = 0; s < 4; s++) {
            if constexpr (F16) nonfinite += f16_nonfinite(gb[s]) ? 1u : 0u;
            adam_element<F16, BC2>(C, gb[s], p[s], m[s], v[s]);
        }
        if (__any(__builtin_isunordered(p[0], p[1]) | __builtin_isunordered(p[2], p[3]))) {
            asm volatile("");  // a branch, not 24 selections in every row
#pragma unroll
            for (int s = 0; s < 4; s++) {
                p[s] = canonical_nan(p[s]);
                m[s] = canonical_nan(m[s]);
                v[s] = canonical_nan(v[s]);
            }
        }
        uint32_t fw[2], fp[4], fm[4], fv[4];
        fw[0] = F16 ? f32_to_f16_pair(p[0], p[1]) : f32_to_bf16_pair(p[0], p[1]);
        fw[1] = F16 ? f32_to_f16_pair(p[2], p[3]) : f32_to_bf16_pair(p[2], p[3]);
#pragma unroll
        for (int s = 0; s < 4; s++) {
            fp[s] = f32_to_bits(p[s]);
            fm[s] = f32_to_bits(m[s]);
            fv[s] = f32_to_bits(v[s]);
        }
        // the results take the place of the inputs
        q[r].g = u32x2{fw[0], fw[1]};
        q[r].p = u32x4{fp[0], fp[1], fp[2], fp[3]};
        q[r].m = u32x4{fm[0], fm[1], fm[2], fm[3]};
        q[r].v = u32x4{fv[0], fv[1], fv[2], fv[3]};
    });
    if (!WHOLE) {
        // slots that are not the tile's are zero, but for the edge elements, which sit in lanes 0..7
        const uint32_t ex[4] = {edge_w, f32_to_bits(ep), f32_to_bits(em), f32_to_bits(ev)};
        static_for<kRows>([&](auto r) {
            const int x = r * kRowElems + 4 * lane;
            if (!mine(r)) q[r] = RowIn{u32x2{0, 0}, u32x4{0, 0, 0, 0}, u32x4{0, 0, 0, 0}, u32x4{0, 0, 0, 0}};
            static_for<2>([&](auto e) {
                uint32_t h[4][4];
                static_for<4>([&](auto i) {
                    static_for<4>([&](auto k) { h[i][k] = __builtin_amdgcn_readlane(ex[i], 4 * e + k); });
                });
                if ((e == 0 ? lo_cut : hi_cut) && x == (e == 0 ? edge_lo : edge_hi)) {
                    q[r].g = u32x2{h[0][0] | (h[0][1] << 16), h[0][2] | (h[0][3] << 16)};
                    q[r].p = u32x4{h[1][0], h[1][1], h[1][2], h[1][3]};
                    q[r].m = u32x4{h[2][0], h[2][1], h[2][2], h[2][3]};
                    q[r].v = u32x4{h[3][0], h[3][1], h[3][2], h[3][3]};
                }
            });
        });
    }
    // Stores from registers, stream by stream; but the fp32 streams of a workgroup that is all at this tile
    // may go by way of its image in LDS (C.image).
    auto store_w = [&](uint8_t* base) {
        static_for<kRows>([&](auto r) {
            if (mine(r)) store8_unaligned<true>(base + (lane8 + 2 * kRowElems * r), q[r].g);
        });
        if (!WHOLE && has_edge)
            *as_global(reinterpret_cast<uint16_t*>(base + 2 * ej)) = static_cast<uint16_t>(edge_w);
    };
    auto store_f = [&](uint8_t* base, u32x4 RowIn::*x, float e) {
        static_for<kRows>([&](auto r) {
            if (mine(r)) store16_unaligned<true>(base + (lane16 + 4 * kRowElems * r), q[r].*x);
        });
        if (!WHOLE && has_edge)
            *as_global(reinterpret_cast<u32_a2*>(base + 4 * ej)) = f32_to_bits(e);
    };
    __builtin_amdgcn_sched_barrier(0);
    store_w(tw);
    store_w(sw);
    const bool by_image = !CHAINED && C.image && ((info >> 8) & 15u) == kWavesPerBlock;
    if (by_image) {
        uint8_t* const im = img + wave * (kSubElems * 4);  // this wavefront's share of every stream
        static_for<kRows>([&](auto r) {
            *reinterpret_cast<u32x4_alias*>(im + (lane16 + 4 * kRowElems * r)) = q[r].p;
            *reinterpret_cast<u32x4_alias*>(im + kImgF + (lane16 + 4 * kRowElems * r)) = q[r].m;
            *reinterpret_cast<u32x4_alias*>(im + 2 * kImgF + (lane16 + 4 * kRowElems * r)) = q[r].v;
        });
    } else {
        if constexpr (!CHAINED) {
            store_f(tp, &RowIn::p, ep);
            store_f(tm, &RowIn::m, em);
            store_f(tv, &RowIn::v, ev);
        }
        store_f(chunks + (static_cast<int64_t>(t.soff[1]) + 4 * at64), &RowIn::p, ep);
        store_f(chunks + (static_cast<int64_t>(t.soff[2]) + 4 * at64), &RowIn::m, em);
        store_f(chunks + (static_cast<int64_t>(t.soff[3]) + 4 * at64), &RowIn::v, ev);
    }
    __builtin_amdgcn_sched_barrier(0);
    // Split first element: its first two bytes close the previous chunk and must not enter this tile's CRC
    // of that stream.
    const bool head = !WHOLE && t.head_split && at <= 0;
    auto dword = [&](auto r, u32x4 RowIn::*x, auto stream, auto f) -> uint32_t {
        uint32_t d = (q[r].*x)[int(f)];
        if (!WHOLE && head && r * kRowElems + 4 * lane == edge_lo && f == (lo & 3) && (t.head_split >> stream & 1u)) {
            add_head_piece(C, crcs, t, tile, 3 + stream, d & 0xFFFFu);
            d &= 0xFFFF0000u;
        }
        return d;
    };
    // Two streams at a time: the sums of all four would take the registers that a third workgroup on the
    // compute unit needs.
    uint32_t bits = 0;
    {
        QuarterSums w = {}, p = {};
        static_for<kRows>([&](auto r) {
            static_for<2>([&](auto f) {
                const u32x4 k[2] = {lds.half[2 * r + f][0][lane], lds.half[2 * r + f][1][lane]};
                matrix_add(w, k, q[r].g[int(f)]);
            });
            static_for<4>([&](auto f) {
                const u32x4 k[2] = {lds.wide[4 * r + f][0][lane], lds.wide[4 * r + f][1][lane]};
                matrix_add(p, k, dword(r, &RowIn::p, std::integral_constant<int, 1>{}, f));
            });
            __builtin_amdgcn_sched_barrier(0);
        });
        matrix_take(bits, w);
        matrix_take(bits, p);
    }
    __builtin_amdgcn_sched_barrier(0);
    {
        QuarterSums m = {}, v = {};
        static_for<kRows>([&](auto r) {
            static_for<4>([&](auto f) {
                const u32x4 k[2] = {lds.wide[4 * r + f][0][lane], lds.wide[4 * r + f][1][lane]};
                matrix_add(m, k, dword(r, &RowIn::m, std::integral_constant<int, 2>{}, f));
                matrix_add(v, k, dword(r, &RowIn::v, std::integral_constant<int, 3>{}, f));
                if (f % 2) __builtin_amdgcn_sched_barrier(0);
            });
        });
        matrix_take(bits, m);
        matrix_take(bits, v);
    }
    const uint32_t reg = row_xor(matrix_streams(bits, lane_c0, lane_c));
    if (WARM && C.tally)
        deliver_to_tally(C, lds, t, info, reg, f, run_entry, crcs, lane);
    else
        deliver(C, lds, t, info, reg, run_entry, crcs, lane);

    if (by_image) {
        workgroup_barrier();
        constexpr int kAll = kWavesPerBlock * int(kSubElems);
        const int from = at - wave * int(kSubElems);
        const int end = static_cast<int>(t.n) - from;
        store_image(t, img, from, from < 0 ? -from : 0, end < kAll ? end : kAll, chunks, wave, lane);
    }

    if constexpr (F16) {
        if (C.n_nonfinite && (__any(nonfinite != 0) || edge_nonfinite)) {
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) nonfinite += __shfl_xor(nonfinite, d);
            nonfinite += edge_nonfinite;
            if (lane == 0) {
                if (C.tally) open_count(C.state, C.epoch, C.n_nonfinite);
                atomicAdd(reinterpret_cast<unsigned long long*>(C.n_nonfinite),
                          static_cast<unsigned long long>(nonfinite));
            }
        }
    }
}

// ---- RAW sub-block: plain copy into the snapshot -------------------------------------------------
//
// Rows are aligned to the stream, so the stores go to whole lines; bytes [lo, hi) of the sub-block
// are the tile's, and its first byte is `at` bytes behind the tile's first (perhaps before it).  A
// slot of 16 bytes that is the tile's only in part is moved halfword by halfword, by lanes 0-7 (the
// slot that holds lo) and 8-15 (the one that holds hi), and handed to its owner for the CRC.
template <bool WARM>
__device__ __forceinline__ void raw_sub_block(const WorkTile& t, const uint32_t info, const int at,
                                              const int lo, const int hi, uint8_t* __restrict__ chunks,
                                              uint32_t* __restrict__ crcs, const FusedConsts& C,
                                              const uint32_t run_entry, Lds& lds,
                                              const uint32_t* __restrict__ lane_tab, int wave, int lane)
{
    const int sub = info & 15u;
    // x^(8 * bytes between the end of the lane's slot and the end of the block)
    const uint32_t to_block_end = lane_tab[(3 - sub) * 64 + lane];
    const uint8_t* const src = reinterpret_cast<const uint8_t*>(t.ptr[0]) + at;
    uint8_t* const dst = chunks + (static_cast<int64_t>(t.soff[0]) + at);
    auto mine = [&](int r) {
        const int x = r * 1024 + 16 * lane;
        return x >= lo && x + 16 <= hi;
    };
    u32x4 w[kRawRows];
    static_for<kRawRows>([&](auto r) {
        w[r] = u32x4{0, 0, 0, 0};
        if (mine(r)) w[r] = load16_unaligned<!WARM>(src + r * 1024 + 16 * lane);
    });
    const int edge_lo = lo & ~15, edge_hi = hi & ~15;
    const bool lo_cut = (lo & 15) || edge_lo + 16 > hi, hi_cut = (hi & 15) && edge_hi > edge_lo;
    uint32_t eh = 0;
    if (lane < 16) {
        const int x = (lane < 8 ? edge_lo : edge_hi) + 2 * (lane & 7);
        if ((lane < 8 ? lo_cut : hi_cut) && x >= lo && x < hi) {
            eh = *as_global(reinterpret_cast<const uint16_t*>(src + x));
            *as_global(reinterpret_cast<uint16_t*>(dst + x)) = static_cast<uint16_t>(eh);
        }
    }
    // and on to the end of the chunk: the wavefronts of a run may be at different tiles of it.  (While the
    // data is on its way.)
    const uint32_t lane_c = gf2_mul(to_block_end, t.shift[0]);
    tables_ready();
    u32x4 edge[2];  // the two slots, put together from the halfwords of lanes 0..15
    static_for<2>([&](auto e) {
        uint32_t h[8];
        static_for<8>([&](auto k) { h[k] = __builtin_amdgcn_readlane(eh, 8 * e + k); });
        edge[e] = u32x4{h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
    });
    uint32_t bits = 0;
    static_for<kRawRows / 2>([&](auto pair) {  // two rows are a stream
        QuarterSums sums = {};
        static_for<2>([&](auto k) {
            constexpr int r = 2 * pair + k;
            const int x = r * 1024 + 16 * lane;
            if (mine(r)) store16_stream<true>(dst + x, w[r]);
            if (lo_cut && x == edge_lo) w[r] = edge[0];
            if (hi_cut && x == edge_hi) w[r] = edge[1];
            static_for<4>([&](auto f) {
                const u32x4 weights[2] = {lds.wide[4 * k + f][0][lane], lds.wide[4 * k + f][1][lane]};
                matrix_add(sums, weights, w[r][int(f)]);
            });
            __builtin_amdgcn_sched_barrier(0);
        });
        matrix_take(bits, sums);
    });
    // (With a run for every tile tensors of 2 KB are bound by the atomics on their chunk's word: 40 MB of
    // them in chunks of 16 KiB / 1 MiB / 8 MiB 49 / 188 / 256 us, with runs across tiles 48 / 52 / 52.)
    uint32_t v = wave_xor(gf2_mul(matrix_share(bits, lane), lane_c));
    if (lane != 0) return;
    const uint32_t run = (info >> 4) & 7u, len = (info >> 8) & 15u;
    if (len > 1 && !run_complete(lds.raw_sum[run], wave - run, len, v)) return;
    if (C.tally)
        add_to_tally(C, run_ticket(C, run_entry, 0), crcs, t.chunk[0], v);
    else
        atomicXor(&crcs[t.chunk[0]], v);
}

// The buffer's end, workgroup by workgroup, and the counter.
constexpr int kTailSlots = 8 * kThreads;
__device__ __forceinline__ void clear_tail(const FusedConsts& C, uint8_t* __restrict__ chunks, const uint32_t part)
{
    const uint64_t first = (C.payload + 15) & ~uint64_t(15);  // chunks is 16-byte aligned, payload even
    if (part == 0) {
        if (threadIdx.x < (first - C.payload) / 2) reinterpret_cast<uint16_t*>(chunks + C.payload)[threadIdx.x] = 0;
        if (threadIdx.x == kThreads - 1 && C.n_nonfinite) open_count(C.state, C.epoch, C.n_nonfinite);
    }
    u32x4* const slots = reinterpret_cast<u32x4*>(chunks + first);
    const uint64_t n = (C.buffer_bytes - first) / 16;
    static_for<kTailSlots / kThreads>([&](auto i) {
        const uint64_t j = uint64_t(part) * kTailSlots + i * kThreads + threadIdx.x;
        if (j < n) slots[j] = u32x4{0, 0, 0, 0};
    });
}

// The gradient pointers of the parameter groups [grad_base, grad_base + kGradsPerLaunch) travel by
// value in the kernel arguments: the step keeps no per-call table in device memory, so calls on
// one plan may overlap and a captured launch carries its own pointers.
//
// N: room for so many.  Arguments of 512 bytes instead of 3 KiB save the host 0.2-0.3 us a call (1 / 8 / 64
// groups 7.4 / 7.9 / 11.0 against 7.7 / 8.1 / 11.2), which shows where a queue of steps is bound by that: 64
// groups of 100 elements 10.7 against 11.2 us a step, fewer or larger groups the same within 1 %; those of 16 KiB
// are for the steps that 3 KiB would cut into several launches.
//
// TALLY: with C.tally or without; else without.  The long chained steps have code of their own, whose 70 registers
// leave a SIMD room for seven wavefronts: still three workgroups, but the next one starts before the last of the third
// is gone.  With the tally's code in it (76 registers, six wavefronts) the first pass of a 7B shard on a new state, when
// every load takes longer, was 1.5 % slower (4952 / 4869 us on one machine, 5026 / 4954 on another), and repeated ones
// 1 % faster (4426-4440 / 4468-4479); 500 ragged parameters 523 / 512, 64 of 600,000 248 / 247.  Two workgroups, made so by
// LDS, 5208 and 4494.  In fp16 seven wavefronts need scratch memory and gain nothing (7B new 5060 with, 5038 without).
template <bool F16, bool CHAINED, bool BC2, uint32_t N, bool TALLY = true>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(TALLY || F16 ? 6 : 7))) void fused_kernel(
    const WorkWave* __restrict__ waves, const WorkTile* __restrict__ tiles, uint32_t grad_base,
    const uint32_t* __restrict__ tabs, uint8_t* __restrict__ chunks, uint32_t* __restrict__ crcs,
    FusedConsts C, GradPtrsOf<N> grads)
{
    __shared__ Lds lds;
    extern __shared__ __attribute__((aligned(16))) uint8_t img[];  // of launches with C.image
    if (!TALLY) C.tally = nullptr;
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWaveSize);
    const uint32_t group = xcd_order(blockIdx.x, gridDim.x, C.xcd_group);
    if (C.tally && group >= C.n_groups) {
        clear_tail(C, chunks, group - C.n_groups);
        return;
    }
    fetch_tables(tabs, lds, wave, lane);
    const WorkWave e = waves[group * kWavesPerBlock + wave];
    const uint32_t run_entry = group * kWavesPerBlock + ((e.info >> 4) & 7u);
    if (e.tile == kNoTile) {
        tables_ready();
        return;
    }
    // the tile descriptor is uniform and read-only: the loads below go through scalar registers
    // (a private copy indexed by the stream number would live in scratch memory instead)
    const WorkTile& t = tiles[e.tile];
    const int sub = e.info & 15u;
    const uint32_t* const lane_tab = tabs + kFusedWeightWords;
    if (t.kind == kWorkRaw) {
        const int at = sub * int(kSubRawBytes) - static_cast<int>(t.soff[0] % kRawTileBytes);
        const int lo = at < 0 ? -at : 0;
        const int left = static_cast<int>(t.n) - at;
        raw_sub_block<false>(t, e.info, at, lo, left < int(kSubRawBytes) ? left : int(kSubRawBytes), chunks,
                      crcs, C, run_entry, lds, lane_tab + 32 * 64, wave, lane);
        return;
    }
    const int at = sub * int(kSubElems) - static_cast<int>(t.e0 % kParamTileElems);
    const int lo = at < 0 ? -at : 0;
    const int left = static_cast<int>(t.n) - at;
    const int hi = left < int(kSubElems) ? left : int(kSubElems);
    const uint8_t* const grad = reinterpret_cast<const uint8_t*>(grads.p[t.grad_index - grad_base]);
    if (lo == 0 && hi == int(kSubElems) && !(t.head_split && at == 0))
        param_sub_block<F16, CHAINED, BC2, true, false>(t, e.tile, e.info, run_entry, at, lo, hi, grad, chunks, crcs, C, lds, img,
                                            lane_tab, wave, lane);
    else
        param_sub_block<F16, CHAINED, BC2, false, false>(t, e.tile, e.info, run_entry, at, lo, hi, grad, chunks, crcs, C, lds, img,
                                             lane_tab, wave, lane);
}

// Steps over small buffers (kWarmStepBytes): they load through the caches; and what the first wavefronts wait for, the
// arguments' lines, then the descriptor's, the gradient's address and the run's tickets, they ask for at once, and the end of the
// chain is shorter (deliver_to_tally).  A kernel of its own, as long steps lose by each: the choice of loads by a branch costs
// lists of 7 million elements and more 3-5 % in place, the earlier start 0.6 % on the 7B shard, chained 0.9 %.
template <bool F16, bool CHAINED, bool BC2, uint32_t N>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(6))) void fused_kernel_warm(
    const WorkWave* __restrict__ waves, const WorkTile* __restrict__ tiles, uint32_t grid,
    const uint32_t* __restrict__ tabs, uint8_t* __restrict__ chunks, uint32_t* __restrict__ crcs,
    FusedConsts C, GradPtrsOf<N> grads)
{
    const uint32_t block = block_behind_args<0, 6 * sizeof(void*) + sizeof(FusedConsts)>();  // up to the gradients'
    __shared__ Lds lds;
    extern __shared__ __attribute__((aligned(16))) uint8_t img[];  // of launches with C.image
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWaveSize);
    const uint32_t group = xcd_order(block, grid, C.xcd_group);
    if (C.tally && group >= C.n_groups) {
        clear_tail(C, chunks, group - C.n_groups);
        return;
    }
    fetch_tables(tabs, lds, wave, lane);
    WorkWave e = waves[group * kWavesPerBlock + wave];
    const uint32_t run_entry = group * kWavesPerBlock + ((e.info >> 4) & 7u);
    if (e.tile == kNoTile) {
        tables_ready();
        return;
    }
    const WorkTile& t = tiles[e.tile];
    const uint64_t grad_at = grads.p[e.info >> 16];
    {
        typedef const __attribute__((address_space(4))) uint32_t Word;
        Word* const words = (Word*)&t;
        Word* const ticket = C.tally ? (Word*)(C.runs + 4 * run_entry) : words;
        const uint32_t all = words[0] | words[16] | words[32] | words[sizeof(WorkTile) / 4 - 1] | *ticket;
        asm("" : "+s"(e.info) : "s"(all), "s"(grad_at));
        __builtin_amdgcn_sched_barrier(0);
    }
    const int sub = e.info & 15u;
    const uint32_t* const lane_tab = tabs + kFusedWeightWords;
    if (t.kind == kWorkRaw) {
        const int at = sub * int(kSubRawBytes) - static_cast<int>(t.soff[0] % kRawTileBytes);
        const int lo = at < 0 ? -at : 0;
        const int left = static_cast<int>(t.n) - at;
        raw_sub_block<true>(t, e.info, at, lo, left < int(kSubRawBytes) ? left : int(kSubRawBytes), chunks,
                      crcs, C, run_entry, lds, lane_tab + 32 * 64, wave, lane);
        return;
    }
    const int at = sub * int(kSubElems) - static_cast<int>(t.e0 % kParamTileElems);
    const int lo = at < 0 ? -at : 0;
    const int left = static_cast<int>(t.n) - at;
    const int hi = left < int(kSubElems) ? left : int(kSubElems);
    const uint8_t* const grad = reinterpret_cast<const uint8_t*>(grad_at);
    if (lo == 0 && hi == int(kSubElems) && !(t.head_split && at == 0))
        param_sub_block<F16, CHAINED, BC2, true, true>(t, e.tile, e.info, run_entry, at, lo, hi, grad, chunks, crcs, C, lds, img,
                                                       lane_tab, wave, lane);
    else
        param_sub_block<F16, CHAINED, BC2, false, true>(t, e.tile, e.info, run_entry, at, lo, hi, grad, chunks, crcs, C, lds, img,
                                                        lane_tab, wave, lane);
}

// ---- the step's traffic alone (bench helper) -------------------------------------------------------
//
// The loads and stores of a parameter tile with no arithmetic and no CRC, in the shape that moved
// this mix of streams fastest in microbenchmarks: a workgroup of 4 wavefronts stages half a tile
// (at most 4096 elements, 56 KiB) in LDS in two phases.  Load: the 1 KiB rows of the four input
// streams -- gradient, master, m, v -- form one list that is cut into four equal runs, and every
// wavefront requests its run up front, so a wavefront sweeps contiguous memory of one or two
// streams.  Store: the rows of the eight output streams -- in place x 4, snapshot x 4 -- form one
// list cut the same way.  The new 16-bit weights are the gradient's bits; master, m, v keep their
// values.  Overlap of loads and stores comes from the two workgroups a CU holds being in different
// phases.  (With the update and the CRC added this shape loses to fused_kernel: a tile must fit
// LDS whole, which halves it, and the per-tile reductions and the update, done in phases of their
// own, then take more ALU time per element than the memory phases leave.)
// Every stream's image in LDS is aligned to its END: a stream of nbytes takes rows = ceil(nbytes /
// 1 KiB) rows and starts pad = rows * 1 KiB - nbytes bytes into its first row.

constexpr int kStageWaves = 4;
constexpr int kStageThreads = kStageWaves * kWaveSize;
constexpr int kStageElems = 4096;
constexpr int kRowsF = kStageElems * 4 / 1024;  // rows of a whole fp32 stream of a half tile
constexpr int kRowsW = kStageElems * 2 / 1024;  // rows of a whole 16-bit stream
constexpr int kRowsIn = kRowsW + 3 * kRowsF;
static_assert(kRowsIn % kStageWaves == 0, "whole half tiles split evenly");
static_assert(kParamTileElems <= 2 * kStageElems, "a parameter tile is staged in two halves");

struct StageGeom {
    int n;               // elements
    int rows_w, rows_f;  // rows of the 16-bit stream / of each fp32 stream
    int pad_w, pad_f;    // bytes in front of the data in row 0
};

// byte offset of stream x's image (0: w16 / gradient, 1..3: master, m, v) in LDS
__device__ __forceinline__ int stage_base(int x)
{
    return x == 0 ? 0 : kRowsW * 1024 + (x - 1) * kRowsF * 1024;
}

template <bool CHAINED>
__global__ __launch_bounds__(kStageThreads) void mix_ceiling_kernel(
    const WorkTile* __restrict__ tiles, uint32_t n_tiles, uint32_t grad_base,
    uint8_t* __restrict__ chunks, FusedConsts C, GradPtrs grads)
{
    __shared__ __attribute__((aligned(16))) uint8_t img[kRowsIn * 1024];
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWaveSize);
    // workgroup position p: half p mod 2 of tile p div 2
    const uint32_t pos = xcd_order(blockIdx.x, gridDim.x, C.xcd_group);
    const uint32_t ti = pos / 2;
    if (ti >= n_tiles) return;
    const WorkTile& t = tiles[ti];
    if (t.kind != kWorkParam) return;
    const int e_off = static_cast<int>(pos % 2) * kStageElems;  // first element of this half
    if (e_off >= static_cast<int>(t.n)) return;
    StageGeom G;
    G.n = static_cast<int>(t.n) - e_off < kStageElems ? static_cast<int>(t.n) - e_off : kStageElems;
    G.rows_w = (2 * G.n + 1023) / 1024;
    G.rows_f = (4 * G.n + 1023) / 1024;
    G.pad_w = G.rows_w * 1024 - 2 * G.n;
    G.pad_f = G.rows_f * 1024 - 4 * G.n;
    const uint32_t lane16 = 16u * lane;
    auto elem_bytes = [](int x) { return x == 0 ? 2 : 4; };

    // ---- load ------------------------------------------------------------------------------------
    {
        // where stream x is read from: the gradient; master, m, v from their tensors or, chained,
        // from the previous snapshot at their stream offsets
        const uint8_t* src[4];
        src[0] = reinterpret_cast<const uint8_t*>(grads.p[t.grad_index - grad_base]) +
                 2 * (t.e0 + e_off);
#pragma unroll
        for (int x = 1; x < 4; x++)
            src[x] = (CHAINED ? C.prev + t.soff[x] : reinterpret_cast<const uint8_t*>(t.ptr[x])) +
                     4 * e_off;
        const int total = G.rows_w + 3 * G.rows_f;
        const int per = (total + kStageWaves - 1) / kStageWaves;
        constexpr int kPer = kRowsIn / kStageWaves;
        u32x4 q[kPer];
        // row i of this wavefront's run: which stream, which row of it (x < 0: none)
        auto decode = [&](int i, int& x, int& r) {
            const int rr = wave * per + i;
            x = -1;
            r = rr;
            if (i < per && rr < total) {
                x = 0;
                if (r >= G.rows_w) {
                    r -= G.rows_w;
                    x = 1;
                    if (r >= G.rows_f) { r -= G.rows_f; x = 2; }
                    if (r >= G.rows_f) { r -= G.rows_f; x = 3; }
                }
            }
        };
        static_for<kPer>([&](auto ic) {
            constexpr int i = ic;
            int x, r;
            decode(i, x, r);
            q[i] = u32x4{0, 0, 0, 0};
            if (x >= 0) {
                const uint8_t* sp = x == 0 ? src[0] : (x == 1 ? src[1] : (x == 2 ? src[2] : src[3]));
                const int pad = x == 0 ? G.pad_w : G.pad_f;
                const int off = r * 1024 + static_cast<int>(lane16) - pad;  // in the stream's data
                if (off >= 0) {
                    q[i] = load16_unaligned<true>(sp + off);
                } else if (off > -16) {
                    // the lane's 16 bytes begin in the pad (row 0 only): halfword by halfword
                    uint32_t h[8];
#pragma unroll
                    for (int u = 0; u < 8; u++) {
                        const int b = off + 2 * u;
                        h[u] = b >= 0 ? *as_global(reinterpret_cast<const uint16_t*>(sp + b)) : 0u;
                    }
                    q[i] = u32x4{h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16),
                                 h[6] | (h[7] << 16)};
                }
            }
        });
        static_for<kPer>([&](auto ic) {
            constexpr int i = ic;
            int x, r;
            decode(i, x, r);
            if (x >= 0) *reinterpret_cast<u32x4*>(&img[stage_base(x) + r * 1024 + lane16]) = q[i];
        });
    }
    __syncthreads();

    // ---- store -----------------------------------------------------------------------------------
    {
        // The output streams in the order their rows are listed: in place master, m, v (not when
        // chained), in place w16, then snapshot master, m, v, w16.  o counts through that list;
        // stream_of(o) is the image it is taken from.
        constexpr int kOut = CHAINED ? 5 : 8;
        constexpr int kInPlace = CHAINED ? 1 : 4;
        auto stream_of = [&](int o) {
            return o < kInPlace ? (o == kInPlace - 1 ? 0 : o + 1) : ((o - kInPlace + 1) & 3);
        };
        auto rows_of = [&](int o) { return stream_of(o) == 0 ? G.rows_w : G.rows_f; };
        const int total = (kOut - 2) * G.rows_f + 2 * G.rows_w;
        const int per = (total + kStageWaves - 1) / kStageWaves;
        constexpr int kPer = 2 * kRowsIn / kStageWaves;
        // this wavefront's run starts at row r of output stream o
        int o = 0, r = wave * per;
        static_for<kOut>([&](auto) {
            if (o < kOut && r >= rows_of(o)) {
                r -= rows_of(o);
                o++;
            }
        });
        static_for<kPer>([&](auto ic) {
            constexpr int i = ic;
            if (i < per && o < kOut) {
                const int x = stream_of(o);
                const int pad = x == 0 ? G.pad_w : G.pad_f;
                uint8_t* const d = (o < kInPlace ? reinterpret_cast<uint8_t*>(t.ptr[x]) : chunks + t.soff[x]) +
                                   elem_bytes(x) * e_off;
                const u32x4 w = *reinterpret_cast<const u32x4*>(&img[stage_base(x) + r * 1024 + lane16]);
                const int off = r * 1024 + static_cast<int>(lane16) - pad;
                if (off >= 0) {
                    store16_unaligned<true>(d + off, w);
                } else if (off > -16) {
                    const uint32_t dd[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
                    for (int u = 0; u < 8; u++) {
                        const int b = off + 2 * u;
                        if (b >= 0)
                            *as_global(reinterpret_cast<uint16_t*>(d + b)) =
                                static_cast<uint16_t>(dd[u >> 1] >> ((u & 1) * 16));
                    }
                }
                r++;
                if (r >= rows_of(o)) {
                    r = 0;
                    o++;
                }
            }
        });
    }
}

// crcs[] = the preset/complement term (the tiles XOR their pieces into it), the tail of the last
// chunk = 0, and the non-finite gradient counter = 0
__global__ void fused_prepare_kernel(uint32_t* __restrict__ crcs, uint64_t n_chunks, uint32_t affine,
                                     uint8_t* __restrict__ chunks, uint64_t payload,
                                     uint64_t buffer_bytes, uint64_t* __restrict__ n_nonfinite)
{
    const uint64_t i = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i == 0 && n_nonfinite) *n_nonfinite = 0;
    const uint64_t stride = static_cast<uint64_t>(gridDim.x) * blockDim.x;
    for (uint64_t j = i; j < n_chunks; j += stride) crcs[j] = affine;
    // the tail: whole 16-byte slots, and the halfwords in front of the first (payload is even)
    const uint64_t first = (payload + 15) & ~uint64_t(15);  // chunks is 16-byte aligned
    if (i < (first - payload) / 2) reinterpret_cast<uint16_t*>(chunks + payload)[i] = 0;
    u32x4* const slots = reinterpret_cast<u32x4*>(chunks + first);
    const uint64_t n_slots = (buffer_bytes - first) / 16;
    for (uint64_t j = i; j < n_slots; j += stride) slots[j] = u32x4{0, 0, 0, 0};
}

}  // namespace

void build_fused_tabs(uint32_t* tab)
{
    for (int r = 0; r < kRows; r++)
        for (int f = 0; f < 4; f++)
            build_quarter_weights(tab + (4 * r + f) * kQuarterWords,
                                  gf2_xpow(8ull * 1024 * (kRows - 1 - r) + 32 * (3 - f)), gf2_xpow(8 * 16 * 16));
    tab += 4 * kRows * kQuarterWords;
    for (int r = 0; r < kRows; r++)
        for (int f = 0; f < 2; f++)
            build_quarter_weights(tab + (2 * r + f) * kQuarterWords,
                                  gf2_xpow(8ull * 512 * (kRows - 1 - r) + 32 * (1 - f)), gf2_xpow(8 * 8 * 16));
    uint32_t* const lane_tab = tab + 2 * kRows * kQuarterWords;
    for (int lane = 0; lane < kWaveSize; lane++) {
        const int quarter = lane / 16, column = lane % 16, stream = quarter;
        uint32_t v;
        for (int wide = 0; wide < 2; wide++) {
            const uint64_t slot = wide ? 16 : 8;
            v = gf2_xpow(8 * slot * (15 - column) + 24 - 8 * quarter);
            const uint32_t x_sub = gf2_xpow(8 * slot * kWaveSize * kRows);
            for (int k = 0; k < 16; k++, v = gf2_mul(v, x_sub)) lane_tab[(16 * wide + k) * 64 + lane] = v;
        }
        v = gf2_xpow(8 * 16 * (15 - column) + 8ull * 2048 * (3 - stream));
        const uint32_t x_raw = gf2_xpow(8ull * kSubRawBytes);
        for (int k = 0; k < 4; k++, v = gf2_mul(v, x_raw)) lane_tab[(32 + k) * 64 + lane] = v;
    }
}

namespace {

constexpr uint32_t kFewGrads = 64, kSomeGrads = 384;

template <uint32_t N>
void launch_step(bool f16, const WorkWave* waves, uint32_t n_waves, const WorkTile* tiles,
                 const void* const* grads, uint32_t p0, uint32_t n_params, const uint32_t* tabs,
                 uint8_t* chunks, uint32_t* crcs, const FusedConsts& consts, bool off_lines, bool warm, hipStream_t stream)
{
    using Kernel = decltype(&fused_kernel<false, false, false, N>);
    static const Kernel kernels[8] = {
        fused_kernel<false, false, false, N>, fused_kernel<false, false, true, N>,
        fused_kernel<false, true, false, N>,  fused_kernel<false, true, true, N>,
        fused_kernel<true, false, false, N>,  fused_kernel<true, false, true, N>,
        fused_kernel<true, true, false, N>,   fused_kernel<true, true, true, N>};
    static const Kernel kernels_warm[8] = {
        fused_kernel_warm<false, false, false, N>, fused_kernel_warm<false, false, true, N>,
        fused_kernel_warm<false, true, false, N>,  fused_kernel_warm<false, true, true, N>,
        fused_kernel_warm<true, false, false, N>,  fused_kernel_warm<true, false, true, N>,
        fused_kernel_warm<true, true, false, N>,   fused_kernel_warm<true, true, true, N>};
    static const Kernel chained[4] = {  // without a tally
        fused_kernel<false, true, false, N, false>, fused_kernel<false, true, true, N, false>,
        fused_kernel<true, true, false, N, false>,  fused_kernel<true, true, true, N, false>};
    const bool bc2 = consts.adam.bc2s != 1.0f;
    const int which = (f16 ? 4 : 0) + (consts.prev ? 2 : 0) + (bc2 ? 1 : 0);
    const Kernel kernel = warm                            ? kernels_warm[which]
                          : consts.prev && !consts.tally ? chained[(f16 ? 2 : 0) + (bc2 ? 1 : 0)]
                                                          : kernels[which];
    // The image only pays in launches of several rounds (aligned, in the one round that there is: 64 parameters
    // of 5000 elements 12.0 us from registers, 13.9 through the image; 32 of 32,768 15.6 and 17.2; 64 of 30,011
    // 23.5 and 23.4) and off the lines (30 odd-sized parameters 2921 from registers, 2700 through it; aligned, 64 of
    // 100,000 58 and 64, 13 of 5 million 514 and 517).
    unsigned groups = n_waves / kWavesPerGroup;
    // (Without those that clear the buffer's end: 760 and 6.6 MB to clear, aligned / off the lines, 26.9 / 31.3 us where
    // they counted, 26.8 / 27.8 where they do not; 732 and 8.1 MB 28.8 / 32.0 and 27.1 / 27.4; 720 and 25 MB 33.7 / 37.0
    // and 34.9 / 35.5.)
    const bool at_once = groups <= 3 * kComputeUnits;
    FusedConsts c = consts;
    if (c.tally) {
        c.n_groups = groups;
        const uint64_t tail = c.buffer_bytes - c.payload;
        groups += static_cast<unsigned>((tail / 16 + kTailSlots - 1) / kTailSlots);
        if (groups == c.n_groups && (tail || c.n_nonfinite)) groups++;
    }
    c.image = !consts.prev && off_lines && !at_once;
    GradPtrsOf<N> g;
    for (uint32_t i = 0; i < N; i++)
        g.p[i] = p0 + i < n_params ? reinterpret_cast<uint64_t>(grads[p0 + i]) : 0;
    hipLaunchKernelGGL(kernel, dim3(groups), dim3(kThreads), consts.prev || at_once ? 0 : c.image ? kImgBytes : kSpareLds, stream, waves,
                       tiles, warm ? groups : p0, tabs, chunks, crcs, c, g);
}

}  // namespace

hipError_t launch_fused(bool f16, const FusedWork& work, const void* const* grads, uint32_t n_params,
                        const uint32_t* tabs, void* chunks, uint32_t* crcs, uint64_t n_chunks,
                        uint64_t payload, uint64_t buffer_bytes, uint32_t affine,
                        const FusedConsts& consts, bool bare, hipStream_t stream)
{
    uint8_t* c = static_cast<uint8_t*>(chunks);
    hipError_t e = hipSuccess;
    if (!bare && !consts.tally) {
        const uint64_t slots = (buffer_bytes - payload) / 16;
        const uint64_t prep_items = n_chunks > slots ? n_chunks : slots;
        unsigned prep_blocks = static_cast<unsigned>((prep_items + 255) / 256);
        if (prep_blocks == 0) prep_blocks = 1;
        if (prep_blocks > 1024) prep_blocks = 1024;
        hipLaunchKernelGGL(fused_prepare_kernel, dim3(prep_blocks), dim3(256), 0, stream, crcs,
                           n_chunks, affine, c, payload, buffer_bytes,
                           f16 ? consts.n_nonfinite : nullptr);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const bool chained = consts.prev != nullptr;
    // one launch per kGradsPerLaunch parameter groups; tiles and wavefronts are sorted by group
    for (uint32_t k = 0, p0 = 0; p0 < n_params; k++, p0 += kGradsPerLaunch) {
        if (bare) {
            const uint32_t t0 = work.launch_tile[k], t1 = work.launch_tile[k + 1];
            if (t1 == t0) continue;
            GradPtrs g;
            for (uint32_t i = 0; i < kGradsPerLaunch; i++)
                g.p[i] = p0 + i < n_params ? reinterpret_cast<uint64_t>(grads[p0 + i]) : 0;
            // two workgroups per tile, one per half
            if (chained)
                hipLaunchKernelGGL(mix_ceiling_kernel<true>, dim3(2 * (t1 - t0)), dim3(kStageThreads),
                                   0, stream, work.tiles + t0, t1 - t0, p0, c, consts, g);
            else
                hipLaunchKernelGGL(mix_ceiling_kernel<false>, dim3(2 * (t1 - t0)),
                                   dim3(kStageThreads), 0, stream, work.tiles + t0, t1 - t0, p0, c, consts,
                                   g);
        } else {
            const uint32_t w0 = work.launch_wave[k], w1 = work.launch_wave[k + 1];
            if (w1 == w0) continue;
            const uint32_t left = n_params - p0;
            const auto launch = left <= kFewGrads    ? launch_step<kFewGrads>
                                : left <= kSomeGrads ? launch_step<kSomeGrads>
                                                     : launch_step<kGradsPerLaunch>;
            launch(f16, work.waves + w0, w1 - w0, work.tiles, grads, p0, n_params, tabs, c, crcs, consts,
                   work.launch_off_lines[k] != 0, buffer_bytes <= kWarmStepBytes, stream);
        }
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return e;
}

}  // namespace ffsnap
