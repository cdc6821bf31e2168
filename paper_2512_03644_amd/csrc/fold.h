// Device-side building blocks shared by the kernels: 16-byte accesses, the table-free CRC
// folding step, and the reduction of a folded state to a 32-bit CRC register.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "fold_taps.h"
#include "gf2.h"

namespace ffsnap {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef u32x4 u32x4_a2 __attribute__((aligned(2)));
typedef u32x2 u32x2_a2 __attribute__((aligned(2)));
typedef uint32_t u32_a2 __attribute__((aligned(2)));

// Every pointer the kernels dereference is device global memory.  Addresses that come out of
// tables are plain integers, so the compiler would fall back to flat (generic) accesses, whose
// completion order it cannot count on; casting to the global address space gives global_load /
// global_store, which complete in order and can be kept in flight with exact wait counts.
#define FF_GLOBAL __attribute__((address_space(1)))
template <class T>
__device__ __forceinline__ FF_GLOBAL T* as_global(T* p)
{
    return (FF_GLOBAL T*)p;
}

constexpr int kWaveSize = 64;

// Barrier of the workgroup for kernels whose wavefronts take different branches (a branch per wavefront,
// never per lane) and come to it in different places of the code.  __syncthreads() may stand only
// where all threads of a workgroup reach the same call; this names what such kernels rely on, and is what
// __syncthreads() compiles to here: s_barrier counts the wavefronts that have arrived, wherever their
// program counters are, and fences on both sides order LDS.  Every wavefront has to execute it the
// same number of times, or end.
__device__ __forceinline__ void workgroup_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// A table of `bytes` on its way into LDS without passing through registers, 16 bytes a lane and load:
// thread t of the workgroup's THREADS fetches slots t, t + THREADS, ...  wait_loads() waits for them.  (Buffer
// loads: next to global loads into LDS the compiler takes no other load's completion for ordered, and
// waits for all of them wherever it waits for one.)
#define FF_LDS __attribute__((address_space(3)))
template <int THREADS, int BYTES>
__device__ __forceinline__ void table_to_lds(const uint32_t* table, u32x4* lds, const int wave, const int lane)
{
    static_assert(BYTES % (16 * THREADS) == 0, "whole rounds");
    constexpr int kWords = 0x00027000;  // of 32 bits, no swizzle
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(table), 0, BYTES, kWords);
    for (int i = 0; i < BYTES / (16 * THREADS); i++)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (FF_LDS void*)(lds + i * THREADS + wave * 64), 16, 16 * lane,
                                                 16 * (i * THREADS + wave * 64), 0, 0);
}
// Until no more than LATER of the loads and stores issued by this wavefront are under way.
template <int LATER>
__device__ __forceinline__ void wait_loads()
{
    static_assert(LATER >= 0 && LATER < 64, "six bits, in two places; the other counters at their largest");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0x0F70 | (LATER & 15) | (LATER >> 4) << 14);
    __builtin_amdgcn_sched_barrier(0);
}

template <class Fn, int... Is>
__device__ __forceinline__ void static_for_impl(Fn&& fn, std::integer_sequence<int, Is...>)
{
    (fn(std::integral_constant<int, Is>{}), ...);
}
template <int N, class Fn>
__device__ __forceinline__ void static_for(Fn&& fn)
{
    static_for_impl(fn, std::make_integer_sequence<int, N>{});
}

// The workgroup's number, known when bytes [FROM, TO) of the kernel's arguments are in the scalar cache.  The compiler
// loads arguments where they are used, and the first wavefronts of a launch wait for memory at every line of them
// that is new, one line after the other; so all are asked for at once.  With the order of the XCDs in closed form and a
// chunk's checksum asked for beforehand, us, before / now: pack of 3 / 32 / 60 MB 9.05 / 14.50 / 23.6 and 8.21 / 14.07 /
// 23.2, verify of 3 / 32 / 100 MB 6.2 / 10.0 / 25.8 and 5.3 / 9.2 / 21.9, pack of 300 MB in tiles 119.5 and 118.4, a skipping
// restore of 20,000 ragged tensors 1151 and 1136.
template <int FROM, int TO>
__device__ __forceinline__ uint32_t block_behind_args()
{
    constexpr int kLine = 64, kFirst = FROM / kLine, kLines = (TO - 1) / kLine - kFirst + 1;
    const auto* const args = (const __attribute__((address_space(4))) uint32_t*)__builtin_amdgcn_kernarg_segment_ptr();
    uint32_t all = 0, block = blockIdx.x;
    static_for<kLines>([&](auto i) { all |= args[(kFirst + i) * (kLine / 4)]; });
    asm("" : "+s"(block) : "s"(all));  // (not volatile: table reads behind it remain scalar loads)
    __builtin_amdgcn_sched_barrier(0);
    return block;
}

// An entry of one of the plan's tables, for the whole wavefront.  By a scalar load, whatever the compiler can tell
// about stores in front of it (open_count): a vector load is done when the rows in front of it are, and the barrier
// waits for it.  By vector / by scalar load, us: restore of 2 / 27 / 40 / 110 MB 6.9 / 9.6 / 16.1 / 43.5 and 6.7 / 9.3 /
// 15.8 / 43.0, of 4 / 112 MB listed 7.5 / 45.9 and 7.2 / 45.7, held blocks of tensors of 5 KiB, 1 GB, 497 and 489.
template <class V>
__device__ __forceinline__ V table_entry(const V* table, const uint32_t i)
{
    return ((const __attribute__((address_space(4))) V*)table)[i];
}

// Tensor side: 16 (or 8) bytes at any even address.  Buffer side: 16-byte aligned.  NT marks
// the access non-temporal (streaming data that will not be reused).
template <bool NT = false>
__device__ __forceinline__ u32x4 load16_unaligned(const uint8_t* p)
{
    if (NT) return __builtin_nontemporal_load(as_global(reinterpret_cast<const u32x4_a2*>(p)));
    return *as_global(reinterpret_cast<const u32x4_a2*>(p));
}
template <bool NT = false>
__device__ __forceinline__ void store16_unaligned(uint8_t* p, u32x4 w)
{
    if (NT)
        __builtin_nontemporal_store(w, as_global(reinterpret_cast<u32x4_a2*>(p)));
    else
        *as_global(reinterpret_cast<u32x4_a2*>(p)) = w;
}
template <bool NT = false>
__device__ __forceinline__ u32x2 load8_unaligned(const uint8_t* p)
{
    if (NT) return __builtin_nontemporal_load(as_global(reinterpret_cast<const u32x2_a2*>(p)));
    return *as_global(reinterpret_cast<const u32x2_a2*>(p));
}
template <bool NT = false>
__device__ __forceinline__ void store8_unaligned(uint8_t* p, u32x2 w)
{
    if (NT)
        __builtin_nontemporal_store(w, as_global(reinterpret_cast<u32x2_a2*>(p)));
    else
        *as_global(reinterpret_cast<u32x2_a2*>(p)) = w;
}
template <bool NT = true>
__device__ __forceinline__ u32x4 load16_stream(const uint8_t* p)
{
    if (NT) return __builtin_nontemporal_load(as_global(reinterpret_cast<const u32x4*>(p)));
    return *as_global(reinterpret_cast<const u32x4*>(p));
}
template <bool NT = true>
__device__ __forceinline__ void store16_stream(uint8_t* p, u32x4 w)
{
    if (NT)
        __builtin_nontemporal_store(w, as_global(reinterpret_cast<u32x4*>(p)));
    else
        *as_global(reinterpret_cast<u32x4*>(p)) = w;
}

// One row into a lane's state.  w[0] is the row's first dword (the highest power).  J counts the
// rows folded since the register rotation was last at zero: physical register row p holds
// logical row (p + J) mod NE.  The dwords that leave the top are XORed into the tap positions
// of the sparse generator multiple F (fold_taps.h).
template <class F, int JJ>
__device__ __forceinline__ void fold_row(uint32_t (&S)[F::NE][F::NF], const uint32_t (&w)[F::NF])
{
    constexpr int NE = F::NE, NF = F::NF, J = JJ % NE;
    constexpr int top = (NE - 1 - J + NE) % NE;  // logical row NE-1 before the shift
    uint32_t t[NF];
    static_for<NF>([&](auto f) { t[f] = S[top][f]; });
    static_for<NF>([&](auto f) { S[top][f] = w[NF - 1 - f]; });  // becomes logical row 0
    static_for<NF>([&](auto f) {
        static_for<F::NTAP>([&](auto k) {
            constexpr int e = F::TAP_E[f][k];
            constexpr int c = F::TAP_F[f][k];
            if constexpr (e != 255) {
                constexpr int p = (e - (J + 1) + 2 * NE) % NE;
                S[p][c] ^= t[f];
            }
        });
    });
}

// a ^ b ^ c in one instruction (the compiler keeps chains of two-operand XORs otherwise).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// a * (a fixed power of x) ^ b with four byte tables (LDS): 4 extractions, 4 lookups, 2 XORs.
__device__ __forceinline__ uint32_t mul_tab_add(const uint32_t* tab, uint32_t a, uint32_t b)
{
    return xor3(xor3(tab[a & 0xFFu], tab[256 + ((a >> 8) & 0xFFu)], tab[512 + ((a >> 16) & 0xFFu)]),
                tab[768 + (a >> 24)], b);
}

// XOR over the 64 lanes, the same value in every lane: inside each row of 16 lanes with DPP moves
// (no LDS round trip as in a shuffle), across the four rows through scalar registers.
__device__ __forceinline__ uint32_t wave_xor(uint32_t v)
{
    v ^= __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true);   // quad_perm [1,0,3,2]: lane ^ 1
    v ^= __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true);   // quad_perm [2,3,0,1]: lane ^ 2
    v ^= __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, true);  // row_half_mirror: the other quad
    v ^= __builtin_amdgcn_mov_dpp(v, 0x140, 0xF, 0xF, true);  // row_mirror: the other eight
    return __builtin_amdgcn_readlane(v, 0) ^ __builtin_amdgcn_readlane(v, 16) ^
           __builtin_amdgcn_readlane(v, 32) ^ __builtin_amdgcn_readlane(v, 48);
}

// One lane per wavefront: adds v to the run's sum in LDS (low half of the word; the high half has a bit for each of
// its wavefronts, `who` of `all`).  True in the wavefront that completes the run; v is then the run's whole sum.
__device__ __forceinline__ bool run_complete(uint64_t& word, const uint32_t who, const uint32_t all, uint32_t& v)
{
    const uint64_t mine = uint64_t(1u << who) << 32 | v;
    const uint64_t now = atomicXor(reinterpret_cast<unsigned long long*>(&word), mine) ^ mine;
    v = static_cast<uint32_t>(now);
    return (now >> 32) == (1u << all) - 1;
}

// State of all lanes -> R / x^32, where R is the CRC register (run from 0) of the rows folded so
// far; the factor x^32 that every register carries is applied once per chunk by the combine
// step.  The result is valid in every lane.  tab: byte tables of x^(8*ROW_BYTES);
// lane_c = x^(8 * (ROW_BYTES/64) * (63 - lane)): lane l sits 63 - l lane widths before the end of
// a row.  XOR3: three-operand XORs.  They shorten the chain by a third; behind a restore that is worth
// 1.2 % (7B shard 3.69 -> 3.65 ms), behind a pack it gains 0.4 % on aligned tensors but loses 1.4 %
// on tensors off the 128-byte lines (1.686 -> 1.711 ms for 5.3 GB), so a pack goes without.
template <class F, bool XOR3>
__device__ __forceinline__ uint32_t reduce_state(const uint32_t (&S)[F::NE][F::NF],
                                                 const uint32_t* tab, uint32_t lane_c)
{
    constexpr int NE = F::NE, NF = F::NF;
    uint32_t acc[NF];
    static_for<NF>([&](auto f) { acc[f] = 0; });
    static_for<NE>([&](auto i) {
        constexpr int e = NE - 1 - i;
        static_for<NF>([&](auto f) {
            if constexpr (XOR3) {
                acc[f] = mul_tab_add(tab, acc[f], S[e][f]);
            } else {
                const uint32_t a = acc[f];
                acc[f] = tab[a & 0xFFu] ^ tab[256 + ((a >> 8) & 0xFFu)] ^
                         tab[512 + ((a >> 16) & 0xFFu)] ^ tab[768 + (a >> 24)] ^ S[e][f];
            }
        });
    });
    uint32_t v = acc[NF - 1];
    static_for<NF - 1>([&](auto i) { v = gf2_mul_const<kX32>(v) ^ acc[NF - 2 - i]; });
    v = gf2_mul(v, lane_c);
#pragma unroll
    for (int l = 0; l < 6; l++) v ^= __shfl_xor(v, 1 << l, kWaveSize);
    return v;
}

}  // namespace ffsnap
