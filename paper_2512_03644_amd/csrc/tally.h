// How the registers of a chunk's tiles or blocks meet in one launch: the tally (kernels.hpp).
#pragma once
#include "fold.h"
#include "kernels.hpp"
#include "matrix_fold.h"

namespace ffsnap {

// The tally of a call (see kernels.hpp for its layout).  Words are 64 bits: what has been summed
// up, and who has contributed.  Every contribution is one returning atomic, so the one that completes
// a word knows it and holds the whole sum; it goes on to the next level alone.
__device__ __forceinline__ uint64_t tally_xor(uint64_t* word, uint32_t bit, uint32_t v)
{
    const uint64_t mine = uint64_t(bit) << 32 | v;
    return atomicXor(reinterpret_cast<unsigned long long*>(word), mine) ^ mine;
}
__device__ __forceinline__ void tally_reset(uint64_t* word)
{
    __hip_atomic_store(word, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The count of damaged chunks without a count of all (T.direct): whoever finds one adds it to *n_bad, which has to
// be zero by then.  Whoever comes first and finds another call's number in the state puts this call's there, sets
// *n_bad to zero and says so; who comes in between waits for that one, which is running and waits for nobody.
// (Numbers are compared for equality only: two host threads may enqueue their calls in another order
// than they got their numbers in.)
__device__ __forceinline__ void open_count(uint64_t* state_word, const uint64_t epoch, uint64_t* n)
{
    unsigned long long* const state = reinterpret_cast<unsigned long long*>(state_word);
    const unsigned long long claimed = 2 * epoch, ready = claimed + 1;
    auto look = [&] { return __hip_atomic_load(state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    for (unsigned long long seen = look();;) {
        if (seen == ready) return;
        if (seen == claimed) {
            __builtin_amdgcn_s_sleep(1);
            seen = look();
            continue;
        }
        const unsigned long long before = atomicCAS(state, seen, claimed);
        if (before == seen) break;
        seen = before;
    }
    const unsigned long long old = atomicExch(reinterpret_cast<unsigned long long*>(n), 0ull);
    asm volatile("" ::"v"(old) : "memory");  // the exchange has been done when its result is here
    __hip_atomic_store(state, ready, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// v: register of one run, at the end of its chunk.  place: of the chunk among the n of this launch.  want: the chunk's
// checksum, of a verdict.
template <int MODE>
__device__ __forceinline__ void tally_run(const TileTables& T, uint32_t v, const uint32_t chunk,
                                          const uint32_t run_index, const uint32_t runs,
                                          const uint32_t place, const uint32_t n, const uint32_t want)
{
    constexpr uint32_t kFan = kTallyFan;
    auto all = [](uint32_t bits) { return bits == 32 ? 0xFFFFFFFFu : (1u << bits) - 1; };
    uint64_t* const groups = T.tally + 1;
    uint64_t* const by_chunk = groups + (T.n_chunks + kFan - 1) / kFan;
    uint32_t bit = run_index, bits = runs;
    if (runs > kFan) {
        uint64_t* const w = by_chunk + T.n_chunks + uint64_t(chunk) * (runs / kFan) + run_index / kFan;
        const uint64_t now = tally_xor(w, 1u << (run_index % kFan), v);
        if ((now >> 32) != all(kFan)) return;  // runs per chunk is a power of two
        tally_reset(w);
        v = static_cast<uint32_t>(now);
        bit = run_index / kFan;
        bits = runs / kFan;
    }
    if (bits > 1) {
        const uint64_t now = tally_xor(by_chunk + chunk, 1u << bit, v);
        if ((now >> 32) != all(bits)) return;
        tally_reset(by_chunk + chunk);
        v = static_cast<uint32_t>(now);
    }
    v ^= T.affine;
    if (MODE == kPack) {
        T.acc[chunk] = v;
        return;
    }
    const uint32_t is_bad = v != want ? 1u : 0u;
    T.acc[chunk] = is_bad;
    if (T.verdict)
        __hip_atomic_store(T.verdict + chunk, verdict_word(T.epoch, is_bad), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (T.direct) {
        if (!is_bad) return;
        if (!T.n_bad_add) open_count(T.state, T.epoch, T.n_bad);
        atomicAdd(reinterpret_cast<unsigned long long*>(T.n_bad), 1ull);
        return;
    }
    // how many chunks are done (low half) and how many of them are bad (high half)
    auto count = [](uint64_t* w, uint32_t bad) {
        const uint64_t mine = uint64_t(bad) << 32 | 1u;
        return atomicAdd(reinterpret_cast<unsigned long long*>(w), mine) + mine;
    };
    const uint32_t n_groups = (n + kFan - 1) / kFan, g = place / kFan;
    uint32_t n_bad = is_bad;
    if (n_groups > 1) {
        const uint64_t now = count(groups + g, n_bad);
        if (static_cast<uint32_t>(now) != (g + 1 < n_groups ? kFan : n - g * kFan)) return;
        tally_reset(groups + g);
        n_bad = static_cast<uint32_t>(now >> 32);
    }
    const uint64_t now = count(T.tally, n_bad);
    if (static_cast<uint32_t>(now) != (n_groups > 1 ? n_groups : n)) return;
    tally_reset(T.tally);
    *T.n_bad = (T.n_bad_add ? *T.n_bad : 0) + (now >> 32);
}

// The chunk's verdict, if its word has it: 2 sound, 3 damaged, 0 none yet.
__device__ __forceinline__ uint32_t look_for_verdict(const uint64_t* word, const uint64_t epoch)
{
    const uint64_t v = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return __builtin_amdgcn_readfirstlane(v == verdict_word(epoch, 0) ? 2u : v == verdict_word(epoch, 1) ? 3u : 0u);
}
// The same when it is there; 0 if patience ends.
__device__ __forceinline__ uint32_t await_verdict(const TileTables& T, const uint32_t chunk)
{
    for (uint32_t n = 0; n < T.polls; n++) {
        if (const uint32_t verdict = look_for_verdict(T.verdict + chunk, T.epoch)) return verdict;
        __builtin_amdgcn_s_sleep(8);  // 512 clocks
    }
    return 0;
}

// The verdict by one wavefront alone, who tells the others.  All that wait for a chunk come here at about the same
// time, so each goes on looking: the first to be through ends the work of all, and workgroups of the chunk that start
// later find its verdict when they come.  (When every workgroup of a chunk read all of it whatever the others had found,
// one row under way at a time, a restore without patience took 50.5 ms for 200 MB in chunks of 32 MiB and 16.3 for 64 MB
// in chunks of 16 MiB; now 0.18 and 0.03, or 21 and 9 where no verdict but theirs comes at all.)
// at: the chunk, n blocks of 8 KiB; weight: of the rows of a block, in LDS; lane_c: the lane's factor in a block;
// AHEAD: rows under way at a time.
template <int AHEAD>
__device__ __forceinline__ uint32_t find_verdict(uint64_t* word, const uint64_t epoch, const uint32_t* want,
                                                 const uint32_t affine, const FF_LDS u32x4* weight, const uint8_t* at,
                                                 const uint32_t n, const uint32_t lane_c, const int lane)
{
    constexpr uint32_t kXBlock = gf2_xpow(8ull * kBlockBytes);
    constexpr int kBlockRows = kBlockBytes / 1024;
    uint32_t from = 16u * lane;
    asm volatile("" : "+v"(from));  // or addresses would be worked out ahead, by every wavefront
    const uint8_t* p = at + from;
    uint32_t reg = 0;
#pragma unroll 1
    for (uint32_t b = 0; b < n; b++) {
        if (const uint32_t verdict = look_for_verdict(word, epoch)) return verdict;
        f32x16 acc = {};
#pragma unroll 1
        for (int r0 = 0; r0 < kBlockRows; r0 += AHEAD, p += 1024 * AHEAD) {
            u32x4 w[AHEAD];
            static_for<AHEAD>([&](auto r) { w[r] = load16_stream<false>(p + 1024 * r); });
            static_for<AHEAD>([&](auto r) {
                static_for<4>([&](auto f) { matrix_add(acc, weight[(4 * (r0 + r) + f) * kWaveSize + lane], w[r][int(f)]); });
                __builtin_amdgcn_sched_barrier(0);  // (the weights of one row at a time)
            });
        }
        reg = gf2_mul_const<kXBlock>(reg) ^ wave_xor(gf2_mul_half(matrix_halves(acc), lane_c));
    }
    const uint32_t is_bad = (gf2_mul_const<kX32>(reg) ^ affine) != *want ? 1u : 0u;
    if (lane == 0)  // what the tally's last will store there
        __hip_atomic_store(word, verdict_word(epoch, is_bad), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return 2u | __builtin_amdgcn_readfirstlane(is_bad);
}

}  // namespace ffsnap
