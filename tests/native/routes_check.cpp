// Host-only check of which kernels a call enqueues, and which of them use the plan's tally.  The
// library's host code runs on a recording stand-in for the HIP runtime: device memory is host memory,
// a launch is noted with its kernel's name and arguments and not run.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <type_traits>
#include <vector>

#include "fused.hpp"
#include "kernels.hpp"
#include "layout.hpp"

using namespace ffsnap;

struct Launch {
    std::string kernel;
    TileTables t;
    hipStream_t stream;
    size_t spare_lds;
    uint32_t groups, image;
    FusedConsts step;  // of the optimizer step
};
static std::vector<Launch> g_log;
// (filled by the objects' constructors, before this file's own)
static std::map<const void*, std::string>& names() { static std::map<const void*, std::string> m; return m; }
static int g_units = 256;  // compute units
static hipStreamCaptureStatus g_capture = hipStreamCaptureStatusNone;
static struct { dim3 g, b; size_t s; hipStream_t q; } g_config;

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char* name, const char*, unsigned, void*, void*, dim3*, dim3*, int*) { names()[f] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, hipStream_t q) { g_config = {g, b, s, q}; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, hipStream_t* q) { *g = g_config.g; *b = g_config.b; *s = g_config.s; *q = g_config.q; return hipSuccess; }
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3, void** args, size_t lds, hipStream_t q)
{
    Launch l{names()[f], TileTables(), q, lds, grid.x, 0, FusedConsts()};
    if (l.kernel.find("fused_kernel") != std::string::npos) {
        l.step = *static_cast<FusedConsts*>(args[6]);
        l.image = l.step.image;
    }
    if (l.kernel.find("block_kernel") != std::string::npos) l.t = *static_cast<TileTables*>(args[0]);
    if (l.kernel.find("tile_kernel") != std::string::npos) l.t = *static_cast<TileTables*>(args[5]);
    g_log.push_back(l);
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = g_units; return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { *p = malloc(n); return hipSuccess; }
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void**, const void*) { return hipErrorNotFound; }
const char* hipGetErrorString(hipError_t) { return "stand-in"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* st) { *st = g_capture; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = nullptr; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
}

#define CHECK(x) do { if (!(x)) { printf("line %d, checked from line %d: %s\n", __LINE__, g_line, #x); exit(1); } } while (0)
static int g_line = 0;
#define FROM_HERE(x) do { g_line = __LINE__; x; } while (0)

static bool is(const Launch& l, const char* part) { return l.kernel.find(part) != std::string::npos; }

// A plan over `n` tensors of `bytes` bytes each, and the outputs of its calls.
struct Job {
    ff_plan* plan = nullptr;
    alignas(16) char chunks[16];
    uint32_t crcs[4], bad[4];
    uint64_t n_bad;
    Job(uint64_t n, uint64_t bytes, uint64_t chunk, uint32_t flags = 0, uint64_t misaligned = 0)
    {
        std::vector<ff_segment> segs;
        for (uint64_t i = 0; i < n; i++)
            segs.push_back({reinterpret_cast<void*>((1ull << 40) + misaligned + i * ((bytes + 255) / 128 * 128)), bytes, FF_BF16, FF_KIND_RAW, 0, 0});
        CHECK(ff_snapshot_plan(segs.data(), n, chunk, flags, &plan) == FF_OK);
    }
    ~Job() { ff_plan_destroy(plan); }
    std::vector<Launch> pack(void* s) { g_log.clear(); CHECK(ff_pack(plan, chunks, crcs, s) == FF_OK); return g_log; }
    std::vector<Launch> restore(uint32_t flags, void* s) { g_log.clear(); CHECK(ff_restore(plan, chunks, crcs, bad, &n_bad, flags, s) == FF_OK); return g_log; }
    std::vector<Launch> listed(uint32_t flags, void* s)
    {
        const uint64_t ids[2] = {0, 1};
        g_log.clear();
        CHECK(ff_restore_chunks(plan, chunks, crcs, ids, 2, bad, &n_bad, flags, s) == FF_OK);
        return g_log;
    }
    std::vector<Launch> to_host(void* s) { g_log.clear(); CHECK(ff_pack_to_host(plan, chunks, crcs, chunks, crcs, 1, s, s) == FF_OK); return g_log; }
};

// The registers of a call meet in the caller's array between a preset and, for a verdict, a finishing
// kernel; no launch of the call knows the tally.
static void check_without_tally(const std::vector<Launch>& log, bool verdict)
{
    bool preset = false, folded = false, finished = false;
    for (const Launch& l : log) {
        CHECK(l.t.tally == nullptr);
        if (is(l, "preset")) preset = true;
        if (l.t.acc) { CHECK(preset); folded = true; }
        if (is(l, "finish_verify")) { CHECK(folded); finished = true; }
    }
    CHECK(folded && finished == verdict);
}
// One launch sums up and delivers.
static void check_with_tally(const std::vector<Launch>& log)
{
    for (const Launch& l : log) {
        CHECK(!is(l, "preset") && !is(l, "finish"));
        CHECK((l.t.acc != nullptr) == (l.t.tally != nullptr));
    }
    CHECK(!log.empty() && log[0].t.tally);
}

static void every_call_without_tally(Job& j, void* s)
{
    check_without_tally(j.pack(s), false);
    check_without_tally(j.to_host(s), false);
    for (uint32_t flags : {0u, FF_RESTORE_VERIFY_ONLY, FF_RESTORE_SKIP_BAD}) {
        check_without_tally(j.restore(flags, s), true);
        check_without_tally(j.listed(flags, s), true);
    }
}
static void every_call_with_tally(Job& j)
{
    check_with_tally(j.pack(nullptr));
    check_with_tally(j.to_host(nullptr));
    for (uint32_t flags : {0u, FF_RESTORE_VERIFY_ONLY, FF_RESTORE_SKIP_BAD}) {
        check_with_tally(j.restore(flags, nullptr));
        check_with_tally(j.listed(flags, nullptr));
    }
}

// A handle says nothing about the queue behind it once its stream may have been destroyed with work in
// flight and the handle given to another, so the tally belongs to the one stream that is never destroyed.
static void only_the_default_stream_uses_the_tally()
{
    for (const bool default_first : {false, true}) {
        Job j(4, 1 << 20, 1 << 16);
        if (default_first) FROM_HERE(every_call_with_tally(j));
        for (void* s : {reinterpret_cast<void*>(0x7f0012340000ull), static_cast<void*>(hipStreamPerThread),
                        static_cast<void*>(hipStreamLegacy), reinterpret_cast<void*>(0x7f0012340000ull)})
            FROM_HERE(every_call_without_tally(j, s));
        FROM_HERE(every_call_with_tally(j));  // whoever called before
        g_capture = hipStreamCaptureStatusActive;
        FROM_HERE(every_call_without_tally(j, nullptr));
        g_capture = hipStreamCaptureStatusNone;
    }
}

// Where the tally costs more than the launches it saves: tiles smaller than a block, verdicts on more than
// 6144 chunks (a pack counts no chunks and keeps it).
static void tally_where_it_pays()
{
    for (uint64_t chunk : {1024, 2048, 4096}) {
        Job j(4, 1 << 20, chunk);
        FROM_HERE(every_call_without_tally(j, nullptr));
    }
    Job fine(4, 1 << 20, 1 << 17, FF_PLAN_TILE_LOG2(12));
    FROM_HERE(check_without_tally(fine.pack(nullptr), false));
    FROM_HERE(check_without_tally(fine.restore(0, nullptr), true));
    FROM_HERE(check_without_tally(fine.listed(0, nullptr), true));
    for (uint32_t flags : {0u, FF_PLAN_TILE_LOG2(13)}) {
        Job last(6144, 8192, 8192, flags), more(6145, 8192, 8192, flags);
        for (uint32_t f : {0u, FF_RESTORE_VERIFY_ONLY, FF_RESTORE_SKIP_BAD}) {
            FROM_HERE(check_with_tally(last.restore(f, nullptr)));
            FROM_HERE(check_without_tally(more.restore(f, nullptr), true));
            FROM_HERE(check_with_tally(more.listed(f, nullptr)));
        }
        FROM_HERE(check_with_tally(more.pack(nullptr)));
    }
}

// The kernel that folds: of a pack and a restore (the scatter of a skipping one), and of a read-only pass.
static const char* folding(const std::vector<Launch>& log)
{
    for (const Launch& l : log)
        if (l.t.acc) return is(l, "block_kernel") ? "blocks" : is(l, "tile_kernel") ? "tiles" : "?";
    return "none";
}
static void blocks_by_size_and_layout()
{
    const std::string blocks = "blocks", tiles = "tiles";
    struct { uint64_t mb, chunk, misaligned; uint32_t flags; std::string moving, reading; } cases[] = {
        {112, 1 << 20, 0, 0, blocks, blocks},        // small
        {112, 1 << 20, 6, 0, blocks, blocks},
        {113, 1 << 20, 0, 0, tiles, blocks},         // medium, on the lines
        {192, 1 << 20, 0, 0, tiles, blocks},
        {192, 1 << 20, 6, 0, blocks, blocks},        // medium, off the lines
        {192, 1 << 20, 64, 0, blocks, blocks},
        {192, 1 << 14, 0, 0, blocks, blocks},        // no room for 32 KiB
        {193, 1 << 20, 0, 0, tiles, tiles},          // large
        {193, 1 << 20, 6, 0, tiles, tiles},
        {113, 1 << 20, 0, FF_PLAN_TILE_LOG2(15), tiles, tiles},  // a tile size that is asked for is kept
        {8, 1 << 20, 6, FF_PLAN_TILE_LOG2(15), tiles, tiles},
        {193, 1 << 20, 0, FF_PLAN_TILE_LOG2(13), blocks, tiles},
    };
    for (const auto& c : cases) {
        Job j(1, c.mb << 20, c.chunk, c.flags, c.misaligned);
        for (void* s : {static_cast<void*>(nullptr), reinterpret_cast<void*>(0x7f0012340000ull)}) {
            g_line = static_cast<int>(c.mb);
            CHECK(folding(j.pack(s)) == c.moving);
            CHECK(folding(j.restore(0, s)) == c.moving);
            CHECK(folding(j.restore(FF_RESTORE_VERIFY_ONLY, s)) == c.reading);
            const auto skip = j.restore(FF_RESTORE_SKIP_BAD, s);
            CHECK(folding(skip) == c.reading);
            CHECK(is(skip.back(), c.moving == blocks ? "block_kernel" : "tile_kernel"));
            CHECK(folding(j.listed(0, s)) == blocks);
        }
    }
}

// The optimizer step: three workgroups on a compute unit for a launch of up to 768, else two; results through
// an image in LDS for a longer launch that is mostly off the lines; neither for a chained step.
static void step_by_size_and_alignment()
{
    struct { uint64_t n, numel, misaligned; bool off; } cases[] = {
        {64, 32768, 0, false}, {96, 32768, 0, false}, {97, 32768, 0, false}, {400, 32768, 0, false},
        {64, 32768, 4, true}, {97, 32768, 4, true}, {97, 32768, 64, true}, {97, 32769, 0, true}, {1000, 5, 4, true},
    };
    for (const auto& c : cases) {
        std::vector<ff_segment> segs;
        std::vector<const void*> grads(c.n, reinterpret_cast<void*>(1ull << 41));
        uint64_t at = (1ull << 40) + c.misaligned;
        for (uint32_t i = 0; i < c.n; i++)
            for (uint32_t kind = FF_KIND_W16; kind <= FF_KIND_V; kind++) {
                const bool w16 = kind == FF_KIND_W16;
                segs.push_back({reinterpret_cast<void*>(at), (w16 ? 2 : 4) * c.numel, w16 ? FF_BF16 : FF_F32, kind, i, 0});
                at += (4 * c.numel + 255) / 256 * 256;
            }
        ff_plan* plan = nullptr;
        CHECK(ff_snapshot_plan(segs.data(), segs.size(), 1 << 20, 0, &plan) == FF_OK);
        const ff_adam_hparams hp = {1e-3f, 0.9f, 0.95f, 1e-8f, 0.1f, 1};
        alignas(16) static char chunks[16], prev_end[16];
        uint32_t crcs[1];
        for (const bool chained : {false, true}) {
            g_log.clear();
            const char* prev = prev_end + (1ull << 33);  // far away; never touched
            CHECK((chained ? ff_adam_step_chained(plan, grads.data(), &hp, 1.0f, nullptr, prev, chunks, crcs, nullptr)
                           : ff_adam_step_snapshot(plan, grads.data(), &hp, chunks, crcs, nullptr)) == FF_OK);
            int launches = 0;
            for (const Launch& l : g_log) {
                if (!is(l, "fused_kernel")) continue;
                launches++;
                g_line = static_cast<int>(c.n);
                CHECK((l.spare_lds != 0) == (!chained && l.groups > 768));
                CHECK((l.image != 0) == (!chained && l.groups > 768 && c.off));
            }
            CHECK(launches == static_cast<int>((c.n + kGradsPerLaunch - 1) / kGradsPerLaunch));
        }
        ff_plan_destroy(plan);
    }
}

// A verdict is known by the number of its call, which every call of a plan advances though few write verdicts: no two
// numbers may look the same in a word, and none like a word that has never been written.
static void verdicts_of_two_calls_differ()
{
    Job j(4, 1 << 20, 1 << 16);
    const auto log = j.restore(FF_RESTORE_SKIP_BAD, nullptr);
    CHECK(log.size() == 1 && log[0].t.verdict && log[0].t.epoch > 0);
    using Word = std::remove_reference_t<decltype(*log[0].t.verdict)>;
    for (const uint64_t later : {1ull, 1ull << 30, 1ull << 31, 1ull << 32, 1ull << 40})
        for (const uint64_t bad : {0, 1})
            for (const uint64_t bad_later : {0, 1}) {
                const Word a = static_cast<Word>(verdict_word(log[0].t.epoch, bad));
                const Word b = static_cast<Word>(verdict_word(log[0].t.epoch + later, bad_later));
                CHECK((a | 1) != (b | 1));
                CHECK(static_cast<Word>(verdict_word(later, bad)) > 1);
            }
    for (uint64_t i = 0; i < 16; i++) CHECK(log[0].t.verdict[i] == 0);  // of the plan's chunks, from the start
}

// A restore that leaves damaged chunks out is one launch where the workgroups of a chunk can be in flight together: no
// more of them than the device has compute units, the whole chip's 256 or a partition's.
static void one_pass_where_a_chunk_fits_the_device()
{
    struct { int units; uint64_t mb, chunk; uint32_t flags; bool one; } cases[] = {
        {256, 100, 16 << 20, 0, true},  {256, 100, 32 << 20, 0, false},   // blocks
        {256, 400, 32 << 20, 0, true},  {256, 400, 64 << 20, 0, false},   // tiles
        {128, 100, 8 << 20, 0, true},   {128, 100, 16 << 20, 0, false},  {128, 400, 16 << 20, 0, true}, {128, 400, 32 << 20, 0, false},
        {32, 100, 2 << 20, 0, true},    {32, 100, 4 << 20, 0, false},    {32, 400, 4 << 20, 0, true},   {32, 400, 8 << 20, 0, false},
        {304, 100, 16 << 20, 0, true},  {304, 100, 32 << 20, 0, false},
    };
    for (const auto& c : cases) {
        g_units = c.units;
        Job j(1, c.mb << 20, c.chunk, c.flags, 6);
        g_line = static_cast<int>(c.mb * 1000 + c.units);
        const auto log = j.restore(FF_RESTORE_SKIP_BAD, nullptr);
        CHECK((log.size() == 1) == c.one);
        CHECK(is(log[0], "kernel_held") == c.one);
        CHECK(c.one || is(log.back(), "block_kernel") || is(log.back(), "tile_kernel"));
    }
    g_units = 256;
}

// The flags may take the place of the checksums that they are found with.  A wavefront that holds a chunk may look at
// its checksum after another has written the flag, so such a restore takes two passes.
static void flags_in_place_of_the_checksums()
{
    for (const uint64_t mb : {8, 400}) {
        Job j(1, mb << 20, 1 << 20);
        g_line = static_cast<int>(mb);
        CHECK(j.restore(FF_RESTORE_SKIP_BAD, nullptr).size() == 1);
        g_log.clear();
        CHECK(ff_restore(j.plan, j.chunks, j.crcs, j.crcs, &j.n_bad, FF_RESTORE_SKIP_BAD, nullptr) == FF_OK);
        CHECK(g_log.size() > 1);
        for (const Launch& l : g_log) CHECK(!is(l, "kernel_held"));
    }
}

// Groups of parameters for the optimizer step, w16, master, m, v of each, and RAW tensors behind them.
struct Step {
    ff_plan* plan = nullptr;
    std::vector<const void*> grads;
    alignas(16) char chunks[16];
    uint32_t crcs[1];
    uint64_t n_nonfinite;
    uint32_t half;
    Step(uint64_t n, uint64_t numel, uint64_t chunk, uint64_t misaligned = 0, uint32_t half = FF_BF16, uint64_t n_raw = 0)
        : grads(n, reinterpret_cast<void*>(1ull << 41)), half(half)
    {
        std::vector<ff_segment> segs;
        uint64_t at = (1ull << 40) + misaligned;
        for (uint32_t i = 0; i < n; i++)
            for (uint32_t kind = FF_KIND_W16; kind <= FF_KIND_V; kind++) {
                const bool w16 = kind == FF_KIND_W16;
                segs.push_back({reinterpret_cast<void*>(at), (w16 ? 2 : 4) * numel, w16 ? half : FF_F32, kind, i, 0});
                at += (4 * numel + 255) / 256 * 256;
            }
        for (uint64_t i = 0; i < n_raw; i++) segs.push_back({reinterpret_cast<void*>(at + (i << 12)), 1000, FF_BF16, FF_KIND_RAW, 0, 0});
        CHECK(ff_snapshot_plan(segs.data(), segs.size(), chunk, 0, &plan) == FF_OK);
    }
    ~Step() { ff_plan_destroy(plan); }
    std::vector<Launch> run(bool chained, void* s)
    {
        const ff_adam_hparams hp = {1e-3f, 0.9f, 0.95f, 1e-8f, 0.1f, 1};
        const char* prev = chunks + (1ull << 40);  // far away; never touched
        g_log.clear();
        CHECK((chained ? ff_adam_step_chained(plan, grads.data(), &hp, 1.0f, half == FF_F16 ? &n_nonfinite : nullptr, prev, chunks, crcs, s)
               : half == FF_F16 ? ff_adam_step_snapshot_f16(plan, grads.data(), &hp, 1.0f, &n_nonfinite, chunks, crcs, s)
                                : ff_adam_step_snapshot(plan, grads.data(), &hp, chunks, crcs, s)) == FF_OK);
        return g_log;
    }
};

// How a step's workgroups share a compute unit hangs on how many of them there are, not on how much of the last chunk
// is left to clear.
static void room_by_the_working_groups()
{
    for (const uint64_t chunk : {1ull << 16, 8ull << 20, 64ull << 20})
        for (const uint64_t misaligned : {0, 4})
            for (const uint64_t n : {150, 191, 193, 250}) {  // of four workgroups each
                Step j(n, 16384, chunk, misaligned);
                g_line = static_cast<int>(n);
                for (void* s : {static_cast<void*>(nullptr), reinterpret_cast<void*>(0x7f0012340000ull)}) {
                    const Launch l = j.run(false, s).back();
                    CHECK((l.spare_lds != 0) == (4 * n > 768));
                    CHECK((l.image != 0) == (4 * n > 768 && misaligned));
                    CHECK(j.run(true, s).back().spare_lds == 0);
                }
            }
}

// The step's kernel: of a short step, and of a long one with or without the code of the tally.
static const char* step_kernel(const Launch& l)
{
    const bool is_short = is(l, "fused_kernel_warmILb"), is_long = is(l, "fused_kernelILb");
    CHECK(is_short != is_long);
    if (is_short) return "short";
    CHECK(is(l, "ELb0EEEv") != is(l, "ELb1EEEv"));
    return is(l, "ELb0EEEv") ? "long, no tally" : "long";
}
// ... hangs on the buffer's size, 80 MiB or more, and on whether a long chained step has a tally.
static void step_kernel_by_size()
{
    void* const named = reinterpret_cast<void*>(0x7f0012340000ull);
    struct { uint64_t n, numel, chunk; bool is_short; } cases[] = {
        {10, 30011, 1 << 18, true},
        {1, 5991862, 1 << 20, true}, {1, 5991863, 1 << 20, false},  // 80 and 81 MiB
        {2049, 2900, 1 << 14, true}, {2049, 2930, 1 << 14, false},  // two launches
        {3, 5000, 1 << 27, false},                                  // one chunk of 128 MiB
    };
    for (const auto& c : cases)
        for (const uint32_t half : {FF_BF16, FF_F16})
            for (const bool chained : {false, true})
                for (void* s : {static_cast<void*>(nullptr), named}) {
                    g_line = static_cast<int>(&c - cases);
                    Step j(c.n, c.numel, c.chunk, 4, half);
                    CHECK((ff_plan_buffer_bytes(j.plan) <= 80ull << 20) == c.is_short);
                    int n = 0;
                    for (const Launch& l : j.run(chained, s)) {
                        if (!is(l, "fused_kernel")) continue;
                        n++;
                        CHECK((l.step.tally != nullptr) == (!s && c.n <= kGradsPerLaunch));
                        const std::string want = c.is_short ? "short" : chained && !l.step.tally ? "long, no tally" : "long";
                        CHECK(step_kernel(l) == want);
                    }
                    CHECK(n == (c.n > kGradsPerLaunch ? 2 : 1));
                }
}

// A step is one launch that sums up in the plan's tally on the default stream, eager, where it is short, its gradients
// are one launch's and no chunk has more contributions than the tally's words take.  Else it knows no tally, and a
// kernel in front of it presets the checksums, clears the buffer's end and counter.
static void step_in_one_launch()
{
    void* const named = reinterpret_cast<void*>(0x7f0012340000ull);
    auto one = [](const std::vector<Launch>& log) {
        CHECK(log.size() == 1 && is(log[0], "fused_kernel"));
        const FusedConsts& c = log[0].step;
        CHECK(step_kernel(log[0]) != std::string("long, no tally"));
        CHECK(c.tally && c.runs && c.heads && c.state && c.epoch && c.affine);
        CHECK(c.n_groups && c.n_groups <= log[0].groups);
        // every 64 KiB behind the payload has a workgroup, and the counter has one in any case
        CHECK((log[0].groups - c.n_groups) * 65536ull >= c.buffer_bytes - c.payload);
        CHECK(log[0].groups > c.n_groups || (c.buffer_bytes == c.payload && !c.n_nonfinite));
        return c.epoch;
    };
    auto several = [](const std::vector<Launch>& log, size_t n) {
        CHECK(log.size() == n + 1 && is(log[0], "fused_prepare"));
        for (size_t i = 1; i <= n; i++) CHECK(is(log[i], "fused_kernel") && !log[i].step.tally && !log[i].step.state);
    };
    for (const uint32_t half : {FF_BF16, FF_F16})
        for (const bool chained : {false, true}) {
            Step j(10, 30011, 1 << 18, 4, half, 7);
            uint64_t before = 0;
            for (int i = 0; i < 3; i++) {
                g_line = __LINE__;
                const uint64_t epoch = one(j.run(chained, nullptr));
                CHECK(epoch > before);
                before = epoch;
            }
            for (void* s : {named, static_cast<void*>(hipStreamPerThread), static_cast<void*>(hipStreamLegacy)})
                FROM_HERE(several(j.run(chained, s), 1));
            for (const auto st : {hipStreamCaptureStatusActive, hipStreamCaptureStatusInvalidated}) {
                g_capture = st;
                FROM_HERE(several(j.run(chained, nullptr), 1));
                FROM_HERE(several(j.run(chained, named), 1));
            }
            g_capture = hipStreamCaptureStatusNone;
            FROM_HERE(one(j.run(chained, nullptr)));
        }
    for (const bool chained : {false, true}) {
        FROM_HERE(one(Step(640, 16384, 1 << 20).run(chained, nullptr)));         // 2560 workgroups
        FROM_HERE(several(Step(641, 16384, 1 << 20).run(chained, nullptr), 1));
        FROM_HERE(one(Step(2048, 5, 1 << 14).run(chained, nullptr)));            // gradients of one launch
        FROM_HERE(several(Step(2049, 5, 1 << 14).run(chained, nullptr), 2));
        FROM_HERE(one(Step(1, 1024 * 4096, 64 << 20).run(chained, nullptr)));    // contributions to one chunk
        FROM_HERE(several(Step(1, 1025 * 4096, 64 << 20).run(chained, nullptr), 1));
    }
}

// A restore that leaves damaged chunks out is one launch by the rules of held_in_one_pass, both sides of each: on the
// default stream, eager, with tiles large enough for a tally.
static void skipping_restore_in_one_pass()
{
    const uint32_t t13 = FF_PLAN_TILE_LOG2(13), t14 = FF_PLAN_TILE_LOG2(14), t15 = FF_PLAN_TILE_LOG2(15);
    struct { uint64_t n, bytes, chunk, misaligned; uint32_t flags; bool one; } cases[] = {
        {1, 112ull << 20, 1 << 20, 0, 0, true},          // small: blocks
        {1, 113ull << 20, 1 << 20, 0, 0, false},         // medium, on the lines: verified in blocks, scattered in tiles
        {1, 192ull << 20, 1 << 20, 0, 0, false},
        {1, 192ull << 20, 1 << 20, 6, 0, true},          // medium, off the lines: blocks
        {1, 193ull << 20, 1 << 20, 0, 0, true},          // large: tiles
        {1, 193ull << 20, 1 << 20, 6, 0, true},
        {100000, 2560, 1 << 20, 6, 0, true},             // large, crowded: blocks
        {1, 100ull << 20, 1 << 20, 0, t15, true},        // tiles that are asked for
        {1, 150ull << 20, 1 << 20, 0, t15, true},
        {1, 192ull << 20, 1 << 20, 0, t13, true},        // blocks that are asked for
        {1, 193ull << 20, 1 << 20, 0, t13, false},
        {1, 20ull << 20, 1 << 20, 0, t14, false},        // neither
        {1, 20ull << 20, 1 << 20, 0, FF_PLAN_TILE_LOG2(12), false},
        {1, 20ull << 20, 1 << 12, 0, 0, false},
        {6144, 8192, 8192, 0, 0, true},                  // words of the tally for so many chunks
        {6145, 8192, 8192, 0, 0, false},
        {1, 400ull << 20, 1 << 15, 0, 0, true},          // in tiles any number
        {1, 400ull << 20, 1 << 20, 0, FF_PLAN_CACHE_HINT(3), true},
        {1, 400ull << 20, 1 << 20, 0, FF_PLAN_CACHE_HINT(1), false},
        {1, 400ull << 20, 1 << 18, 0, 0, true},          // 1600 chunks of 256 KiB: two passes have a kernel of their own
    };
    for (const auto& c : cases) {
        Job j(c.n, c.bytes, c.chunk, c.flags, c.misaligned);
        for (void* s : {static_cast<void*>(nullptr), reinterpret_cast<void*>(0x7f0012340000ull), static_cast<void*>(hipStreamPerThread)})
            for (const auto capture : {hipStreamCaptureStatusNone, hipStreamCaptureStatusActive}) {
                g_capture = capture;
                g_line = static_cast<int>(&c - cases);
                const bool one = c.one && !s && capture == hipStreamCaptureStatusNone;
                const auto log = j.restore(FF_RESTORE_SKIP_BAD, s);
                CHECK((log.size() == 1) == one);
                CHECK(is(log[0], "kernel_held") == one);
                if (one) {
                    CHECK(log[0].t.verdict && log[0].t.epoch && log[0].t.polls && log[0].t.tally && log[0].t.want && !log[0].t.skip_bad);
                    CHECK((log[0].t.direct != 0) == (is(log[0], "block_kernel") && log[0].t.n_chunks <= kDirectChunks));
                } else {
                    for (const Launch& l : log) CHECK(!is(l, "kernel_held") && !l.t.verdict);
                    const TileTables& last = log.back().t;
                    CHECK(last.skip_bad == j.bad && !last.acc && !last.tally);
                }
            }
        g_capture = hipStreamCaptureStatusNone;
        for (const uint32_t flags : {0u, FF_RESTORE_VERIFY_ONLY, FF_RESTORE_VERIFY_ONLY | FF_RESTORE_SKIP_BAD})
            for (const Launch& l : j.restore(flags, nullptr)) CHECK(!is(l, "kernel_held"));
        for (const Launch& l : j.listed(FF_RESTORE_SKIP_BAD, nullptr)) CHECK(!is(l, "kernel_held"));
    }
}

// Runs of the XCDs' order: short in restores and in packs in blocks of more than 80 MiB, up to 4 GiB, unless the flags name one.
static void order_by_size()
{
    const uint32_t rule = kDefaultXcdGroup, brief = kShortXcdGroup;
    struct { uint64_t n, bytes, misaligned; uint32_t flags, pack, restore; } cases[] = {
        {1, 80ull << 20, 0, 0, rule, rule},
        {1, 81ull << 20, 0, 0, brief, brief},              // blocks
        {1, 192ull << 20, 0, 0, rule, brief},              // tiles
        {1, 192ull << 20, 6, 0, brief, brief},             // blocks
        {1, 4096ull << 20, 0, 0, rule, brief},
        {1, 4097ull << 20, 0, 0, rule, rule},
        {100000, 2560, 6, 0, brief, brief},                // blocks, whatever the size
        {200000, 2560, 6, 0, 2 * brief, 2 * brief},
        {1, 100ull << 20, 0, FF_PLAN_XCD_ORDER(7), 64, 64},
        {1, 100ull << 20, 0, FF_PLAN_XCD_ORDER(31), 0, 0},
    };
    for (const auto& c : cases) {
        Job j(c.n, c.bytes, 1 << 20, c.flags, c.misaligned);
        g_line = static_cast<int>(&c - cases);
        CHECK(j.pack(nullptr).back().t.xcd_group == c.pack);
        CHECK(j.restore(0, nullptr)[0].t.xcd_group == c.restore);
        const uint32_t given = c.flags ? c.pack : rule;
        CHECK(j.restore(FF_RESTORE_VERIFY_ONLY, nullptr)[0].t.xcd_group == given);
        CHECK(j.listed(0, nullptr)[0].t.xcd_group == given);  // 2 MiB of it
    }
}

// The caches that a pass in blocks goes through: warm up to 96 MiB; a restore of small tensors through them again above 896 MiB.
static void caches_by_size()
{
    const uint32_t around = 3, mid = FF_PLAN_TILE_LOG2(13);
    struct { uint64_t n, bytes, misaligned; uint32_t flags, restore; } cases[] = {
        {1, 96ull << 20, 0, 0, kHintWarm(kRestore)},
        {1, 97ull << 20, 0, 0, around},
        {100000, 4096, 6, 0, around},                       // 390 MiB, in blocks
        {229376, 4096, 6, 0, around},                       // 896 MiB
        {229377, 4096, 6, 0, 0},
        {229377, 4096, 6, mid, around},                     // blocks that are asked for
        {229377, 4096, 6, FF_PLAN_CACHE_HINT(1), 1},
        {1, 1100ull << 20, 0, 0, around},                   // tiles
    };
    for (const auto& c : cases) {
        Job j(c.n, c.bytes, 1 << 20, c.flags, c.misaligned);
        g_line = static_cast<int>(&c - cases);
        const auto log = j.restore(0, nullptr);
        CHECK(log[0].t.hint == c.restore);
        CHECK(is(log[0], "block_kernel") == (c.n > 1 || c.bytes <= 97ull << 20));
        if (!is(log[0], "block_kernel")) continue;
        CHECK(is(log[0], ("block_kernelILi1ELi" + std::to_string(c.restore) + "E").c_str()));
    }
    // A restore that holds its chunks, or of a list of them, has no kernel that goes through the caches both ways: its tables say
    // what its kernel does.
    auto check = [](const std::vector<Launch>& log, const std::string& part, uint32_t hint) {
        int n = 0;
        for (const Launch& l : log)
            if (is(l, (part + std::to_string(hint) + "E").c_str())) { CHECK(l.t.hint == hint); n++; }
        CHECK(n == 1);
    };
    Job small(300000, 4096, 1 << 20, 0, 6), large(600000, 4096, 1 << 30, 0, 6);
    FROM_HERE(check(small.restore(FF_RESTORE_SKIP_BAD, nullptr), "block_kernel_heldILi", around));
    FROM_HERE(check(small.listed(0, nullptr), "block_kernel_listedILi1ELi", kHintWarm(kRestore)));  // 2 MiB
    FROM_HERE(check(large.listed(0, nullptr), "block_kernel_listedILi1ELi", around));               // 2 GiB
}

int main()
{
    caches_by_size();
    order_by_size();
    step_in_one_launch();
    step_kernel_by_size();
    skipping_restore_in_one_pass();
    room_by_the_working_groups();
    one_pass_where_a_chunk_fits_the_device();
    flags_in_place_of_the_checksums();
    verdicts_of_two_calls_differ();
    step_by_size_and_alignment();
    blocks_by_size_and_layout();
    only_the_default_stream_uses_the_tally();
    tally_where_it_pays();
    printf("ok\n");
    return 0;
}
