#include "layout.hpp"

#include <algorithm>
#include <map>

#include "gf2.h"

namespace ffsnap {

static bool is_pow2(uint64_t v) { return v && !(v & (v - 1)); }

int build_layout(const ff_segment* segs, uint64_t n_segs, uint64_t chunk_bytes, unsigned tile_log2,
                 Layout& L)
{
    if (n_segs && !segs) return FF_ERR_NULL;
    if (!is_pow2(chunk_bytes) || chunk_bytes < FF_MIN_CHUNK_BYTES || chunk_bytes > FF_MAX_CHUNK_BYTES)
        return FF_ERR_INVALID;
    if (n_segs >= 0xFFFFFFFFull) return FF_ERR_INVALID;

    L = Layout();
    L.chunk_bytes = chunk_bytes;
    uint64_t off = 0;
    for (uint64_t i = 0; i < n_segs; i++) {
        const ff_segment& s = segs[i];
        if (s.dtype != FF_BF16 && s.dtype != FF_F32 && s.dtype != FF_F16) return FF_ERR_INVALID;
        if (s.kind > FF_KIND_V || s.reserved != 0) return FF_ERR_INVALID;
        const uint64_t es = (s.dtype == FF_F32) ? 4 : 2;
        if (s.nbytes % es) return FF_ERR_INVALID;
        if (s.nbytes == 0) continue;  // empty segments take no place in the stream
        if (!s.ptr) return FF_ERR_NULL;
        if (reinterpret_cast<uint64_t>(s.ptr) % es) return FF_ERR_INVALID;
        if (off + s.nbytes < off) return FF_ERR_INVALID;
        L.segs.push_back(Seg{reinterpret_cast<uint64_t>(s.ptr), off, s.nbytes, s.dtype, s.kind,
                             s.param_id});
        off += s.nbytes;
    }
    if (off == 0) return FF_ERR_EMPTY;
    L.payload = off;
    L.n_chunks = (off + chunk_bytes - 1) / chunk_bytes;
    L.buffer_bytes = L.n_chunks * chunk_bytes;

    // layout id: CRC32C over (chunk_bytes, nbytes...) as little-endian uint64
    {
        std::vector<uint64_t> key;
        key.reserve(L.segs.size() + 1);
        key.push_back(chunk_bytes);
        for (const Seg& s : L.segs) key.push_back(s.nbytes);
        L.layout_id = crc32c_host(key.data(), key.size() * sizeof(uint64_t));
    }

    // parameter groups
    {
        std::map<uint32_t, Param> groups;
        bool ok = true;
        for (size_t i = 0; i < L.segs.size(); i++) {
            const Seg& s = L.segs[i];
            if (s.kind == FF_KIND_RAW) continue;
            auto it = groups.find(s.param_id);
            if (it == groups.end())
                it = groups.emplace(s.param_id, Param{s.param_id, {-1, -1, -1, -1}, 0}).first;
            int32_t& slot = it->second.seg[s.kind - 1];
            if (slot >= 0) ok = false;  // the same role twice
            slot = static_cast<int32_t>(i);
            // working weights are 16-bit, of one format throughout the plan; the rest is fp32
            if (s.kind == FF_KIND_W16) {
                if (s.dtype == FF_F32) ok = false;
                if (L.half_dtype == 0) L.half_dtype = s.dtype;
                if (s.dtype != L.half_dtype) ok = false;
            } else if (s.dtype != FF_F32) {
                ok = false;
            }
        }
        for (auto& kv : groups) {
            Param& p = kv.second;
            bool complete = p.seg[0] >= 0 && p.seg[1] >= 0 && p.seg[2] >= 0 && p.seg[3] >= 0;
            if (!complete) { ok = false; continue; }
            p.numel = L.segs[p.seg[1]].nbytes / 4;
            if (L.segs[p.seg[0]].nbytes != 2 * p.numel || L.segs[p.seg[2]].nbytes != 4 * p.numel ||
                L.segs[p.seg[3]].nbytes != 4 * p.numel)
                ok = false;
            L.params.push_back(p);
        }
        L.adam_ok = ok;
        if (!ok) L.params.clear();
    }

    // tiling
    auto cut_tiles = [&](uint64_t tile) {
        L.tile_bytes = tile;
        L.tiles_per_chunk = static_cast<uint32_t>(chunk_bytes / tile);
        L.n_tiles = L.buffer_bytes / tile;
        L.tile_first_seg.resize(L.n_tiles);
        size_t si = 0;
        for (uint64_t k = 0; k < L.n_tiles; k++) {
            const uint64_t s = k * tile;
            while (si + 1 < L.segs.size() && L.segs[si].off + L.segs[si].nbytes <= s) si++;
            L.tile_first_seg[k] = static_cast<uint32_t>(si);
        }
    };
    uint64_t tile = kDefaultTileBytes;
    if (tile_log2) tile = 1ull << std::min<unsigned>(std::max<unsigned>(tile_log2, 10), 30);
    auto base_of = [&](uint64_t k) -> uint64_t {  // address of tile k if it lies inside one segment, else 0
        const uint64_t s = k * L.tile_bytes;
        const Seg& g = L.segs[L.tile_first_seg[k]];
        return g.off <= s && s + L.tile_bytes <= g.off + g.nbytes ? g.ptr + (s - g.off) : 0;
    };
    cut_tiles(std::min(tile, chunk_bytes));
    if (!tile_log2) {
        uint64_t crowded = 0, on_line = 0;
        for (uint64_t k = 0; k < L.n_tiles; k++) {
            if (k + 1 < L.n_tiles) crowded += L.tile_first_seg[k + 1] - L.tile_first_seg[k] >= 4 ? 1 : 0;
            const uint64_t base = base_of(k);
            on_line += base && base % 128 == 0 ? 1 : 0;
        }
        const bool small = L.buffer_bytes <= kSmallBufferBytes;
        const bool medium = L.buffer_bytes <= kMediumBufferBytes &&
                            (L.tile_bytes < kDefaultTileBytes || on_line < L.n_tiles / 2);
        if (small || medium || crowded > L.n_tiles / kCrowdedShare)
            cut_tiles(std::min(kSmallTileBytes, chunk_bytes));
    }
    L.tile_base.resize(L.n_tiles);
    for (uint64_t k = 0; k < L.n_tiles; k++) L.tile_base[k] = base_of(k);
    return FF_OK;
}

namespace {

// x has order 2^31 - 1 modulo the generator (a primitive polynomial of degree 31 times x + 1), so
// exponents can be taken modulo that, negative ones too.
constexpr int64_t kOrder = 0x7FFFFFFF;
static_assert(gf2_xpow(kOrder) == kOne, "order of x");

// x^n from one table per byte of the exponent: three multiplications.
struct PowTable {
    uint32_t t[4][256];
    PowTable()
    {
        for (int i = 0; i < 4; i++) {
            const uint32_t base = gf2_xpow(1ull << (8 * i));
            t[i][0] = kOne;
            for (int b = 1; b < 256; b++) t[i][b] = gf2_mul(t[i][b - 1], base);
        }
    }
    uint32_t operator()(int64_t n) const
    {
        const uint32_t e = static_cast<uint32_t>((n % kOrder + kOrder) % kOrder);
        return gf2_mul(gf2_mul(t[0][e & 255], t[1][(e >> 8) & 255]),
                       gf2_mul(t[2][(e >> 16) & 255], t[3][e >> 24]));
    }
};

// The factor that takes the register of a block (without its x^32) whose last byte ends at stream
// offset block_end to the end of chunk `chunk`.
uint32_t shift_to_chunk_end(const PowTable& xp, uint64_t chunk, uint64_t block_end,
                            uint64_t chunk_bytes)
{
    const int64_t d = static_cast<int64_t>((chunk + 1) * chunk_bytes) - static_cast<int64_t>(block_end);
    return xp(32 + 8 * d);
}

}  // namespace

void build_work_tiles(const Layout& L, std::vector<WorkTile>& out)
{
    out.clear();
    const PowTable xp;
    const uint64_t C = L.chunk_bytes;
    std::vector<bool> in_group(L.segs.size(), false);
    for (size_t pi = 0; pi < L.params.size(); pi++) {
        const Param& p = L.params[pi];
        const uint64_t size[4] = {2, 4, 4, 4};
        uint64_t off[4], ptr[4];
        for (int x = 0; x < 4; x++) {
            off[x] = L.segs[p.seg[x]].off;
            ptr[x] = L.segs[p.seg[x]].ptr;
            in_group[p.seg[x]] = true;
        }
        // cut points: (element, streams whose element is split there)
        std::map<uint64_t, uint32_t> cuts;
        cuts[0] = 0;
        for (int x = 0; x < 4; x++) {
            const uint64_t a = off[x], b = off[x] + size[x] * p.numel;
            for (uint64_t B = (a / C + 1) * C; B < b; B += C) {
                const uint64_t e = (B - a) / size[x];
                uint32_t& m = cuts[e];
                if ((B - a) % size[x]) m |= 1u << x;
            }
        }
        for (auto it = cuts.begin(); it != cuts.end(); ++it) {
            auto nx = std::next(it);
            const uint64_t end = (nx == cuts.end()) ? p.numel : nx->first;
            for (uint64_t e0 = it->first; e0 < end;) {
                const uint64_t block_end = (e0 / kParamTileElems + 1) * kParamTileElems;
                WorkTile t{};
                t.kind = kWorkParam;
                t.grad_index = static_cast<uint32_t>(pi);
                t.e0 = e0;
                t.n = static_cast<uint32_t>(std::min(block_end, end) - e0);
                t.head_split = (e0 == it->first) ? it->second : 0;
                for (int x = 0; x < 4; x++) {
                    t.ptr[x] = ptr[x] + size[x] * e0;
                    t.soff[x] = off[x] + size[x] * e0;
                    uint64_t begin = t.soff[x];
                    if (t.head_split & (1u << x)) {
                        t.chunk[3 + x] = static_cast<uint32_t>(begin / C);
                        t.shift[3 + x] = kOne;  // the two head bytes end their chunk
                        begin += 2;
                    }
                    t.chunk[x] = static_cast<uint32_t>(begin / C);
                    t.shift[x] = shift_to_chunk_end(xp, t.chunk[x], off[x] + size[x] * block_end, C);
                }
                out.push_back(t);
                e0 += t.n;
            }
        }
    }
    for (size_t i = 0; i < L.segs.size(); i++) {
        if (in_group[i]) continue;
        const Seg& s = L.segs[i];
        uint64_t pos = 0;
        while (pos < s.nbytes) {
            const uint64_t abs = s.off + pos;
            const uint64_t block_end = (abs / kRawTileBytes + 1) * kRawTileBytes;
            uint64_t len = std::min<uint64_t>(block_end - abs, s.nbytes - pos);
            len = std::min<uint64_t>(len, (abs / C + 1) * C - abs);
            WorkTile t{};
            t.kind = kWorkRaw;
            t.n = static_cast<uint32_t>(len);
            t.ptr[0] = s.ptr + pos;
            t.soff[0] = abs;
            t.chunk[0] = static_cast<uint32_t>(abs / C);
            t.shift[0] = shift_to_chunk_end(xp, t.chunk[0], block_end, C);
            out.push_back(t);
            pos += len;
        }
    }
}

bool build_work_waves(const std::vector<WorkTile>& tiles, uint64_t n_params,
                      uint32_t groups_per_launch, std::vector<WorkWave>& out,
                      std::vector<uint32_t>& begin, uint64_t max_entries)
{
    out.clear();
    begin.assign(1, 0);
    auto fill_group = [&] {
        while (out.size() % kWavesPerGroup) out.push_back(WorkWave{kNoTile, 0});
    };
    const uint64_t launches = (n_params + groups_per_launch - 1) / groups_per_launch;
    for (size_t i = 0; i < tiles.size(); i++) {
        const WorkTile& t = tiles[i];
        uint64_t first, last;  // sub-blocks the tile touches
        if (t.kind == kWorkParam) {
            const uint64_t in_block = t.e0 % kParamTileElems;
            first = in_block / kSubElems;
            last = (in_block + t.n - 1) / kSubElems;
            while (begin.size() <= t.grad_index / groups_per_launch) {
                fill_group();
                begin.push_back(static_cast<uint32_t>(out.size()));
            }
        } else {
            const uint64_t in_block = t.soff[0] % kRawTileBytes;
            first = in_block / kSubRawBytes;
            last = (in_block + t.n - 1) / kSubRawBytes;
        }
        // a tile that fills workgroups gets them to itself
        if (last - first + 1 >= kWavesPerGroup) fill_group();
        for (uint64_t s = first; s <= last;) {
            const uint64_t slot = out.size() % kWavesPerGroup;
            const uint64_t here = std::min<uint64_t>(last - s + 1, kWavesPerGroup - slot);
            // a RAW tile goes on with the run in front of it, if that is of the same chunk
            uint64_t begin = slot, run = here;
            const WorkTile* before = slot && out.back().tile != kNoTile ? &tiles[out.back().tile] : nullptr;
            if (t.kind == kWorkRaw && before && before->kind == kWorkRaw && before->chunk[0] == t.chunk[0]) {
                begin = (out.back().info >> 4) & 7u;
                run = slot + here - begin;
                for (uint64_t k = out.size() - slot + begin; k < out.size(); k++)
                    out[k].info = (out[k].info & 0xFFu) | static_cast<uint32_t>(run << 8);
            }
            const uint32_t grad = t.kind == kWorkParam ? t.grad_index % groups_per_launch : 0;
            for (uint64_t k = 0; k < here; k++, s++)
                out.push_back(WorkWave{static_cast<uint32_t>(i),
                                       static_cast<uint32_t>(s | (begin << 4) | (run << 8)) | grad << 16});
        }
        if (out.size() > max_entries) return false;
    }
    fill_group();
    if (out.size() > max_entries) return false;
    while (begin.size() < launches + 1) begin.push_back(static_cast<uint32_t>(out.size()));
    return true;
}

bool build_step_tickets(const std::vector<WorkTile>& tiles, const std::vector<WorkWave>& waves, uint64_t n_chunks,
                        std::vector<StepTicket>& runs, std::vector<StepTicket>& heads, uint64_t& words)
{
    runs.assign(4 * waves.size(), StepTicket{});
    heads.assign(3 * tiles.size(), StepTicket{});
    std::vector<uint32_t> count(n_chunks, 0);
    // in two passes: a contribution's place in its chunk first (in root, for now), with the chunk in leaf
    auto take = [&](StepTicket& t, uint32_t chunk) {
        t.leaf = chunk;
        t.root = count[chunk]++;
        t.leaf_full = 1;  // taken
    };
    for (size_t i = 0; i < waves.size(); i++) {
        if (waves[i].tile == kNoTile || i % kWavesPerGroup != ((waves[i].info >> 4) & 7u)) continue;
        const WorkTile& t = tiles[waves[i].tile];
        const bool one = t.kind == kWorkRaw ||
                         (t.chunk[0] == t.chunk[1] && t.chunk[0] == t.chunk[2] && t.chunk[0] == t.chunk[3]);
        for (int x = 0; x < (one ? 1 : 4); x++) take(runs[4 * i + x], t.chunk[x]);
    }
    for (size_t i = 0; i < tiles.size(); i++)
        for (int x = 1; x < 4; x++)
            if (tiles[i].kind == kWorkParam && (tiles[i].head_split >> x & 1u)) take(heads[3 * i + x - 1], tiles[i].chunk[3 + x]);
    std::vector<uint32_t> base(n_chunks);
    words = 0;
    for (uint64_t c = 0; c < n_chunks; c++) {
        const uint32_t leaves = (count[c] + 31) / 32;
        if (leaves > 32) return false;
        base[c] = static_cast<uint32_t>(words);
        words += leaves + (leaves > 1 ? 1 : 0);
    }
    auto place = [&](StepTicket& t) {
        if (!t.leaf_full) return;
        const uint32_t chunk = t.leaf, k = t.root, n = count[chunk], leaves = (n + 31) / 32, leaf = k / 32;
        const uint32_t here = leaf + 1 < leaves ? 32 : n - 32 * leaf;
        t.leaf = base[chunk] + leaf;
        t.leaf_full = here == 32 ? 0xFFFFFFFFu : (1u << here) - 1;
        t.bits = k % 32 | leaves << 8 | leaf << 16;
        t.root = base[chunk] + leaves;
    };
    for (StepTicket& t : runs) place(t);
    for (StepTicket& t : heads) place(t);
    return true;
}

bool mostly_off_lines(const WorkTile* tiles, uint64_t n)
{
    uint64_t off = 0, all = 0;
    for (uint64_t i = 0; i < n; i++) {
        const WorkTile& t = tiles[i];
        bool line = true;
        for (int x = 1; x < 4; x++)  // rows begin at multiples of 512 bytes from the parameter's first element
            line = line && (t.ptr[x] - 4 * t.e0) % 128 == 0 && (t.soff[x] - 4 * t.e0) % 128 == 0;
        all += t.n;
        off += line ? 0 : t.n;
    }
    return 2 * off > all;
}

}  // namespace ffsnap
