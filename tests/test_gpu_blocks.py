"""Pack, restore and verify in 8 KiB blocks against the oracle: at the sizes where a block can go
wrong (crowded blocks, slots that straddle boundaries, the payload's end, runs shorter than a
workgroup, every level of the tally), and on every route a call can take -- the tally of the default
stream, other streams without it, a replayed capture, listed chunks of a plan with larger tiles."""
import ctypes
import threading
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from paper_2512_03644_amd import binding as ff
from paper_2512_03644_amd import workloads as wl
from test_gpu_parity import DEV, _host_segments, _pack_and_compare, _poison_segments, \
    _restore_and_compare, _u32

pytestmark = pytest.mark.gpu


def _ragged(n, mu, sigma, seed, chunk, max_numel=1 << 16):
    lay = wl.fragmented_layout(seed=seed, n_tensors=n, mu=mu, sigma=sigma, max_numel=max_numel)
    return wl.fragmented_shard(lay, chunk, seed=seed, device=DEV)


@pytest.mark.parametrize("chunk", [1 << 13, 1 << 14, 1 << 16, 1 << 19, 1 << 20, 1 << 22])
@pytest.mark.parametrize("mu,n", [(0.0, 40000), (2.5, 9000), (5.0, 3000), (8.0, 300)])
def test_blocks_of_small_tensors(oracle, chunk, mu, n):
    # on average 5, 45, 600 and 11000 bytes a tensor: from thousands in a block (beyond the table) to
    # less than one
    shard = _ragged(n, mu, 1.0, int(10 * mu) + chunk % 97, chunk)
    state = _pack_and_compare(shard, oracle)
    _restore_and_compare(shard, *state[:6])


@pytest.mark.parametrize("n_seg", [1, 2, 127, 128, 129, 130])
@pytest.mark.parametrize("end", [2, 14, 16, 18, 8190, 8192])
def test_one_block_of_so_many_tensors(oracle, n_seg, end):
    # a block whose payload ends at `end` bytes, cut into n_seg tensors of odd halfword counts
    cuts = np.linspace(0, 8192 * 2 + end, n_seg + 1).astype(np.int64) // 2
    lay = [(int(b - a), 2, (2 * i) % 16) for i, (a, b) in enumerate(zip(cuts[:-1], cuts[1:])) if b > a]
    shard = wl.fragmented_shard(lay, 1 << 13, seed=n_seg, device=DEV)
    state = _pack_and_compare(shard, oracle, tile_log2=13)
    _restore_and_compare(shard, *state[:6])


# one tensor, a few, around the 64 lanes, around the 128 that the table of a block holds, beyond it
@pytest.mark.parametrize("n_seg", [1, 2, 63, 64, 65, 127, 128, 129, 130, 170])
@pytest.mark.parametrize("behind", [False, True])
@pytest.mark.parametrize("tile_log2", [0, 13, 15])
def test_exactly_so_many_tensors_in_one_block(oracle, n_seg, behind, tile_log2):
    # a tensor that ends where the block begins, then n_seg in the block: all boundaries are inside a slot,
    # each in one of its own, so there are as many straddling slots as there can be.  Behind them the
    # payload ends inside a slot too, or a tensor begins where the next block does.
    sizes = [2] + [48] * (n_seg - 2) if n_seg > 1 else []
    last = (8192 if behind else 8192 - 16 * 3 - 6) - sum(sizes)
    sizes.append(last)
    assert len(sizes) == n_seg and last > 0
    ends = 8192 + np.cumsum(sizes)
    assert all(e % 16 for e in ends[:-1]) and len({e // 16 for e in ends}) == n_seg
    starts = ends - sizes
    assert sum(a < 16384 and e > 8192 for a, e in zip(starts, ends)) == n_seg
    lay = [(4096, 2, 6)] + [(b // 2, 2, (2 * i) % 16) for i, b in enumerate(sizes)]
    if behind:
        lay += [(5000, 2, 10)]
    shard = wl.fragmented_shard(lay, 1 << 15, seed=n_seg, device=DEV)
    state = _pack_and_compare(shard, oracle, tile_log2)
    _restore_and_compare(shard, *state[:6])
    # and as a list of chunks, in blocks whatever the tiles are
    plan, chunks, crcs, bad, n_bad, want_buf, _ = state
    _poison_segments(shard)
    ff.ff_restore_chunks(plan, chunks, crcs, list(range(plan.num_chunks)), bad, n_bad)
    torch.cuda.synchronize()
    assert int(n_bad.item()) == 0
    assert np.array_equal(np.concatenate(_host_segments(shard)[0]), want_buf[:plan.payload_bytes])


# up to four tensors in a block go without its table
@pytest.mark.parametrize("tile_log2", [0, 13, 15, 16])
@pytest.mark.parametrize("sizes", [
    [2, 2, 2], [6, 2, 4, 2], [16, 2, 14], [14, 2, 16], [18, 30, 16], [1022, 2, 1024], [1024, 8, 1016], [1030, 1024, 2042],
    [8190], [8190, 2], [8192, 2], [8186, 4], [2, 8190, 2], [4098, 4094, 8192], [2, 2, 2, 2], [2048, 2, 2, 2], [3000, 3000, 2188],
    [30000], [30000, 2, 2], [40960, 2, 24576]])
def test_blocks_of_a_few_tensors(oracle, sizes, tile_log2):
    # boundaries at the start of a slot, of a row, of a block and inside them, several in one slot, blocks of a larger tile that
    # its first tensors do not reach; behind them a payload that goes on for many blocks, or ends inside a slot
    for front, back in ((4096, 20000), (4096, 3), (4095, 0), (1, 0)):
        lay = [(front, 2, 6)] + [(b // 2, 2, (2 * i) % 16) for i, b in enumerate(sizes)] + ([(back, 2, 10)] if back else [])
        shard = wl.fragmented_shard(lay, 1 << 16, seed=sum(sizes), device=DEV)
        state = _pack_and_compare(shard, oracle, tile_log2)
        _restore_and_compare(shard, *state[:6])
        plan, chunks, crcs, bad, n_bad, want_buf, _ = state
        _poison_segments(shard)
        ff.ff_restore_chunks(plan, chunks, crcs, list(range(plan.num_chunks)), bad, n_bad)
        torch.cuda.synchronize()
        assert int(n_bad.item()) == 0
        assert np.array_equal(np.concatenate(_host_segments(shard)[0]), want_buf[:plan.payload_bytes])


def _verify(plan, chunks, crcs, stream=None, flags=ff.FF_RESTORE_VERIFY_ONLY):
    bad = torch.full((plan.num_chunks,), 7, dtype=torch.int32, device=DEV)
    n_bad = torch.full((1,), 99, dtype=torch.int64, device=DEV)
    torch.cuda.synchronize()
    ff.ff_restore(plan, chunks, crcs, bad, n_bad, flags, stream=stream)
    torch.cuda.synchronize()
    return _u32(bad), int(n_bad.item())


# one run per chunk, several, more than one word of 32 of them; one group of 32 chunks and more
@pytest.mark.parametrize("chunk,n_chunks", [(1 << 13, 7), (1 << 13, 1100), (1 << 16, 33), (1 << 18, 40),
                                            (1 << 22, 9), (1 << 23, 3)])
def test_every_level_of_the_tally_and_the_routes_without_it(oracle, chunk, n_chunks):
    nbytes = chunk * n_chunks - 1026
    shard = wl.fragmented_shard([(nbytes // 2, 2, 2)], chunk, seed=n_chunks, device=DEV)
    plan, chunks, crcs, _, _, want_buf, want_crcs = _pack_and_compare(shard, oracle, tile_log2=13)
    assert plan.num_chunks == n_chunks
    damaged = sorted({0, n_chunks - 1, n_chunks // 2, (5 * n_chunks) // 7})
    for j in damaged:
        chunks[j * chunk + 77 + j % 900] ^= 4
    want = np.zeros(n_chunks, np.uint32)
    want[damaged] = 1
    side = torch.cuda.Stream()
    for _ in range(2):                                       # the tally comes back to zero
        for stream in (None, side):                          # with it, and without
            bad, n_bad = _verify(plan, chunks, crcs, stream)
            assert np.array_equal(bad, want) and n_bad == len(damaged)
    _poison_segments(shard)
    bad, n_bad = _verify(plan, chunks, crcs, None, ff.FF_RESTORE_SKIP_BAD)
    assert np.array_equal(bad, want) and n_bad == len(damaged)
    got = _host_segments(shard)[0][0]
    for j in range(n_chunks):
        a, b = j * chunk, min((j + 1) * chunk, nbytes)
        assert np.array_equal(got[a:b], np.full(b - a, 0xA5, np.uint8) if want[j] else want_buf[a:b])


@pytest.mark.parametrize("mis", [0, 6])
@pytest.mark.parametrize("chunk", [1 << 14, 1 << 15, 1 << 20])
def test_medium_buffers_on_and_off_the_lines(oracle, mis, chunk):
    # 113 MiB: moved in 32 KiB tiles if they lie on the tensors' lines (in chunks that have room), in blocks
    # otherwise, and verified in blocks either way
    n_chunks = (113 << 20) // chunk
    shard = wl.fragmented_shard([(chunk * n_chunks // 2 - 7, 2, mis)], chunk, seed=chunk + mis, device=DEV,
                                max_gap=0)
    assert shard.segments[0].data_ptr() % 128 == mis
    plan, chunks, crcs, bad, n_bad, want_buf, _ = _pack_and_compare(shard, oracle)
    assert plan.num_chunks == n_chunks
    _restore_and_compare(shard, plan, chunks, crcs, bad, n_bad, want_buf)
    damaged = [0, n_chunks // 3, n_chunks - 1]
    for j in damaged:
        chunks[j * chunk + 1029 + j % 900] ^= 2
    want = np.zeros(n_chunks, np.uint32)
    want[damaged] = 1
    for stream in (None, torch.cuda.Stream()):
        for flags in (ff.FF_RESTORE_VERIFY_ONLY, ff.FF_RESTORE_SKIP_BAD):
            _poison_segments(shard)
            got_bad, got_n = _verify(plan, chunks, crcs, stream, flags)
            assert np.array_equal(got_bad, want) and got_n == len(damaged)
            got = _host_segments(shard)[0][0].reshape(-1)
            kept = np.full(got.size, flags == ff.FF_RESTORE_VERIFY_ONLY)
            for j in damaged:
                kept[j * chunk:(j + 1) * chunk] = True
            assert np.array_equal(got, np.where(kept, np.uint8(0xA5), want_buf[:got.size]))


def test_replayed_capture_beside_eager_calls(oracle):
    shard = _ragged(800, 7.0, 1.5, 3, 1 << 16)
    plan, chunks, crcs, bad, n_bad, want_buf, want_crcs = _pack_and_compare(shard, oracle)
    chunks2, crcs2 = torch.empty_like(chunks), torch.empty_like(crcs)
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        ff.ff_pack(plan, chunks2, crcs2, stream=side)
        ff.ff_restore(plan, chunks2, crcs2, bad, n_bad, ff.FF_RESTORE_VERIFY_ONLY, stream=side)
    for _ in range(4):
        chunks.fill_(0), crcs.fill_(0), chunks2.fill_(0), crcs2.fill_(0), bad.fill_(3), n_bad.fill_(3)
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            graph.replay()
        for _ in range(3):
            ff.ff_pack(plan, chunks, crcs)
        torch.cuda.synchronize()
        for c, r in ((chunks, crcs), (chunks2, crcs2)):
            assert np.array_equal(c.cpu().numpy(), want_buf) and np.array_equal(_u32(r), want_crcs)
        assert int(n_bad.item()) == 0 and not _u32(bad).any()


def _hip():
    """The HIP runtime that this process has loaded."""
    maps = {l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l}
    return ctypes.CDLL(sorted(maps)[0])


def test_threads_and_streams_that_come_and_go(oracle):
    # Two host threads on the default stream, two on their per-thread streams, and streams that are
    # destroyed with their work in flight, whose handles the runtime may give to the next one: every call
    # gets its own chunks, checksums and verdicts right.
    shard = _ragged(3000, 8.0, 1.5, 21, 1 << 18)
    plan, chunks, crcs, _, _, want_buf, want_crcs = _pack_and_compare(shard, oracle)
    damaged = chunks.clone()
    damaged[5 * (1 << 18) + 99] ^= 16
    hip = _hip()
    outs = [ff.alloc_outputs(plan, DEV) for _ in range(12)]
    torch.cuda.synchronize()

    def calls(stream, out, times):
        for _ in range(times):
            ff.ff_pack(plan, out[0], out[1], stream=stream)
            ff.ff_restore(plan, damaged, crcs, out[2], out[3], ff.FF_RESTORE_VERIFY_ONLY, stream=stream)

    per_thread = SimpleNamespace(cuda_stream=2)  # hipStreamPerThread
    default = SimpleNamespace(cuda_stream=0)
    workers = [threading.Thread(target=calls, args=(s, outs[k], 20))
               for k, s in enumerate((default, default, per_thread, per_thread))]
    for w in workers:
        w.start()
    for k in range(4, 12):
        handle = ctypes.c_void_p()
        assert hip.hipStreamCreateWithFlags(ctypes.byref(handle), 1) == 0
        calls(SimpleNamespace(cuda_stream=handle.value), outs[k], 5)
        assert hip.hipStreamDestroy(handle) == 0
    for w in workers:
        w.join()
    torch.cuda.synchronize()
    want_bad = np.zeros(plan.num_chunks, np.uint32)
    want_bad[5] = 1
    for c, r, bad, n_bad in outs:
        assert np.array_equal(c.cpu().numpy(), want_buf) and np.array_equal(_u32(r), want_crcs)
        assert np.array_equal(_u32(bad), want_bad) and int(n_bad.item()) == 1


@pytest.mark.parametrize("tile_log2", [13, 14, 15, 17])
@pytest.mark.parametrize("flags", [0, ff.FF_RESTORE_VERIFY_ONLY, ff.FF_RESTORE_SKIP_BAD])
def test_listed_chunks_of_any_plan(oracle, tile_log2, flags):
    # listed chunks go in blocks whatever the plan's tiles are, in launches of 254 chunks
    chunk = 1 << 17
    shard = _ragged(7000, 9.0, 1.5, tile_log2, chunk)
    plan, chunks, crcs, bad, n_bad, want_buf, _ = _pack_and_compare(shard, oracle, tile_log2=tile_log2)
    n = plan.num_chunks
    assert n > 600
    ids = [j for j in range(n) if j % 2 == 0 or j == n - 1]
    damaged = [ids[1], ids[300], ids[-1]]
    for j in damaged:
        chunks[j * chunk + 5] ^= 1
    sent = chunks.cpu().numpy()
    _poison_segments(shard)
    bad.fill_(7)
    n_bad.fill_(99)
    ff.ff_restore_chunks(plan, chunks, crcs, ids, bad, n_bad, flags)
    torch.cuda.synchronize()
    assert int(n_bad.item()) == len(damaged)
    got_bad = _u32(bad)
    assert all(got_bad[j] == (1 if j in damaged else 0 if j in set(ids) else 7) for j in range(n))
    want = np.full(plan.payload_bytes, 0xA5, np.uint8)
    for j in ids:
        if flags == ff.FF_RESTORE_VERIFY_ONLY or (flags == ff.FF_RESTORE_SKIP_BAD and j in damaged):
            continue
        a, b = j * chunk, min((j + 1) * chunk, plan.payload_bytes)
        want[a:b] = sent[a:b]
    assert np.array_equal(np.concatenate(_host_segments(shard)[0]), want)


@pytest.mark.parametrize("chunk,tile_log2", [(1 << 13, 10), (1 << 13, 11), (1 << 13, 12), (1 << 12, 10),
                                             (1 << 14, 11), (1 << 15, 10)])
def test_verify_where_grouped_tiles_are_as_long_as_a_block(oracle, chunk, tile_log2):
    # a read-only pass groups tiles up to 64 KiB or the chunk: groups of 8 KiB are not blocks
    shard = _ragged(60, 8.0, 1.0, tile_log2, chunk)
    plan, chunks, crcs, _, _, _, _ = _pack_and_compare(shard, oracle, tile_log2=tile_log2)
    chunks[3 * chunk + 11] ^= 8
    want = np.zeros(plan.num_chunks, np.uint32)
    want[3] = 1
    for stream in (None, torch.cuda.Stream()):
        bad, n_bad = _verify(plan, chunks, crcs, stream)
        assert np.array_equal(bad, want) and n_bad == 1


@pytest.mark.parametrize("chunk", [1 << 13, 1 << 16])
def test_every_weight_of_the_matrix_product(oracle, chunk):
    # One bit per block: dword d of block d, bit (d / 4) mod 32 of it, so that every bit of every place in a
    # lane's rows comes up in either half of the wavefront.  Then the largest counts: blocks of ones.
    words = np.zeros((2048 + 16, 2048), np.uint32)
    d = np.arange(2048)
    words[d, d] = np.uint32(1) << (d // 4 % 32).astype(np.uint32)
    words[2048:] = 0xFFFFFFFF
    words[2048 + 8, 1000:] = 0
    raw = words.view(np.uint8).reshape(-1)
    t = torch.from_numpy(raw.view(np.int16).copy()).to(DEV).view(torch.bfloat16)
    plan = ff.ff_snapshot_plan([t], chunk, tile_log2=13)
    chunks, crcs, bad, n_bad = ff.alloc_outputs(plan, DEV)
    ff.ff_pack(plan, chunks, crcs)
    ff.ff_restore(plan, chunks, crcs, bad, n_bad)
    torch.cuda.synchronize()
    assert np.array_equal(chunks.cpu().numpy(), raw) and int(n_bad.item()) == 0
    want = [oracle.crc32c(raw[k:k + chunk]) for k in range(0, raw.size, chunk)]
    assert np.array_equal(_u32(crcs), np.array(want, np.uint32))


# Restores that leave damaged chunks out in one pass: tiles inside one tensor on and off the lines, of two to four
# tensors, of more, at the payload's end and behind it; runs of 1, 2, 4 and 8 wavefronts; waits that end at
# once; the routes that take two passes (other streams, larger chunks); more chunks than one word counts.
_HELD = {
    "whole": [(1 << 20, 2, 0), (3 << 18, 2, 0)],
    "off": [(1 << 20, 2, 2), (700001, 4, 12), (1 << 19, 2, 14)],
    "pieces": [(9001 + 7 * i, 2 if i % 3 else 4, (2 * i) % 16 if i % 3 else 4) for i in range(200)],
    "crowded": [(1 << 19, 2, 6)] + [(900 + i, 2, (2 * i) % 16) for i in range(150)] + [(300000, 4, 8)],
}


@pytest.mark.parametrize("layout", list(_HELD))
@pytest.mark.parametrize("chunk_log2", [13, 15, 16, 18, 20, 22])
@pytest.mark.parametrize("tile_log2", [13, 15])
def test_restore_without_damaged_chunks_in_one_pass(oracle, layout, chunk_log2, tile_log2):
    chunk = 1 << chunk_log2
    shard = wl.fragmented_shard(_HELD[layout], chunk, seed=chunk_log2, device=DEV)
    plan, chunks, crcs, _, _, want_buf, _ = _pack_and_compare(shard, oracle, tile_log2=min(tile_log2, chunk_log2))
    n = plan.num_chunks
    damaged = sorted({0, n // 2, n - 1} if n > 3 else {n - 1})
    for j in damaged:
        chunks[j * chunk + (911 * j + 5) % chunk] ^= 64
    want_bad = np.zeros(n, np.uint32)
    want_bad[damaged] = 1
    keep = np.repeat(want_bad != 0, chunk)[:plan.payload_bytes]
    for polls, stream in ((4096, None), (0, None), (4096, torch.cuda.Stream()), (1, None)):
        ff._check(ff.lib().ff_plan_set_polls(plan.handle, polls))
        _poison_segments(shard)
        before = np.concatenate(_host_segments(shard)[0])
        bad, n_bad = _verify(plan, chunks, crcs, stream, ff.FF_RESTORE_SKIP_BAD)
        assert np.array_equal(bad, want_bad) and n_bad == len(damaged)
        got = np.concatenate(_host_segments(shard)[0])
        assert np.array_equal(got, np.where(keep, before, want_buf[:plan.payload_bytes]))


@pytest.mark.parametrize("chunk_log2,nbytes", [(15, 240 << 20), (24, 70 << 20), (25, 200 << 20), (26, 200 << 20)])
def test_one_pass_over_many_and_over_large_chunks(chunk_log2, nbytes):
    # 7680 chunks; chunks of 256 workgroups and of one more than the route takes
    chunk = 1 << chunk_log2
    g = torch.Generator(device=DEV)
    g.manual_seed(chunk_log2)
    t = torch.empty(nbytes // 2 - 1001, dtype=torch.int16, device=DEV).random_(generator=g)
    src = t.clone()
    plan = ff.ff_snapshot_plan([t.view(torch.bfloat16)], chunk)
    chunks, crcs, bad, n_bad = ff.alloc_outputs(plan, DEV)
    ff.ff_pack(plan, chunks, crcs)
    j = plan.num_chunks // 3
    chunks[j * chunk + 12345] ^= 1
    for rep in range(3):
        t.fill_(rep)
        ff.ff_restore(plan, chunks, crcs, bad, n_bad, ff.FF_RESTORE_SKIP_BAD)
        torch.cuda.synchronize()
        assert int(n_bad.item()) == 1 and int(bad.sum().item()) == 1 and int(bad[j].item()) == 1
        want = src.clone()
        want[j * chunk // 2:(j + 1) * chunk // 2] = rep
        assert torch.equal(t, want)


# verdicts counted one by one (128 chunks in a launch) and level by level (more), of which none, some or all are
# damaged, in changing order; lists of more chunks than one launch takes add to the count
@pytest.mark.parametrize("n_chunks", [1, 2, 127, 128, 129, 300])
@pytest.mark.parametrize("chunk_log2", [13, 16])
def test_count_of_damaged_chunks(n_chunks, chunk_log2):
    chunk = 1 << chunk_log2
    g = torch.Generator(device=DEV)
    g.manual_seed(n_chunks)
    t = torch.empty(n_chunks * chunk // 2 - 3, dtype=torch.int16, device=DEV).random_(generator=g)
    plan = ff.ff_snapshot_plan([t.view(torch.bfloat16)], chunk)
    chunks, crcs, bad, n_bad = ff.alloc_outputs(plan, DEV)
    ff.ff_pack(plan, chunks, crcs)
    rng = np.random.default_rng(n_chunks)
    for share in (1.0, 0.0, 0.3, 1.0, 0.02, 0.0):
        hit = np.flatnonzero(rng.random(n_chunks) < share)
        at = torch.from_numpy(hit * chunk + rng.integers(0, chunk, hit.size)).to(DEV)
        chunks[at] ^= 8
        want = np.zeros(n_chunks, np.uint32)
        want[hit] = 1
        for flags in (ff.FF_RESTORE_VERIFY_ONLY, 0, ff.FF_RESTORE_SKIP_BAD):
            bad.fill_(7)
            n_bad.fill_(99)
            ff.ff_restore(plan, chunks, crcs, bad, n_bad, flags)
            torch.cuda.synchronize()
            assert np.array_equal(_u32(bad), want) and int(n_bad.item()) == hit.size
        bad.fill_(7)
        n_bad.fill_(99)
        ff.ff_restore_chunks(plan, chunks, crcs, list(range(n_chunks)), bad, n_bad, ff.FF_RESTORE_VERIFY_ONLY)
        torch.cuda.synchronize()
        assert np.array_equal(_u32(bad), want) and int(n_bad.item()) == hit.size
        chunks[at] ^= 8


def test_pack_of_more_blocks_with_half_the_weights(oracle):
    # one bit in every block of 160 MB, at every place of a block in turn, and tensors that begin anywhere
    n = 20000
    words = torch.zeros((n, 2048), dtype=torch.int32, device=DEV)
    k = torch.arange(n, device=DEV)
    at = k % 2048
    words[k, at] = (torch.ones_like(k) << ((at // 4 + k // 2048) % 31)).to(torch.int32)
    flat = words.view(torch.int16).reshape(-1).view(torch.bfloat16)
    cuts = [0, 700001, 700002, 3000000] + list(range(3100001, 3400000, 1501)) + [flat.numel()]
    segs = [flat[a:b] for a, b in zip(cuts[:-1], cuts[1:])]
    chunk = 1 << 20
    plan = ff.ff_snapshot_plan(segs, chunk, tile_log2=13)
    chunks, crcs, _, _ = ff.alloc_outputs(plan, DEV)
    ff.ff_pack(plan, chunks, crcs)
    torch.cuda.synchronize()
    assert torch.equal(chunks[:plan.payload_bytes], flat.view(torch.uint8)) and not chunks[plan.payload_bytes:].any()
    raw = chunks.cpu().numpy()
    want = [oracle.crc32c(raw[j:j + chunk]) for j in range(0, raw.size, chunk)]
    assert np.array_equal(_u32(crcs), np.array(want, np.uint32))


@pytest.mark.parametrize("chunk_log2,nbytes", [(24, 64 << 20), (25, 200 << 20)])
def test_waits_that_end_at_once_cost_a_chunk_and_not_its_square(chunk_log2, nbytes):
    # blocks, tiles of 32 KiB.  Every workgroup of a chunk reading all of it is 256 times the work (it took 600 times as
    # long); one verdict for all costs each about what it reads until then.
    chunk = 1 << chunk_log2
    t = torch.zeros(nbytes // 2 - 1001, dtype=torch.bfloat16, device=DEV)
    plan = ff.ff_snapshot_plan([t], chunk)
    chunks, crcs, bad, n_bad = ff.alloc_outputs(plan, DEV)
    ff.ff_pack(plan, chunks, crcs)

    def best(polls):
        ff._check(ff.lib().ff_plan_set_polls(plan.handle, polls))
        times = []
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            ff.ff_restore(plan, chunks, crcs, bad, n_bad, ff.FF_RESTORE_SKIP_BAD)
            b.record()
            torch.cuda.synchronize()
            assert int(n_bad.item()) == 0
            times.append(a.elapsed_time(b))
        return min(times)

    assert best(0) < 30 * best(4096)


@pytest.mark.parametrize("nbytes", [8 << 20, 200 << 20])
def test_flags_written_over_the_checksums(nbytes):
    chunk = 1 << 20
    t = torch.arange(nbytes // 2 - 77, dtype=torch.int32, device=DEV).to(torch.int16).view(torch.bfloat16)
    src = t.clone()
    plan = ff.ff_snapshot_plan([t], chunk)
    chunks, crcs, _, n_bad = ff.alloc_outputs(plan, DEV)
    ff.ff_pack(plan, chunks, crcs)
    chunks[3 * chunk + 4321] ^= 2
    t.zero_()
    ff._check(ff.lib().ff_plan_set_polls(plan.handle, 0))
    ff.ff_restore(plan, chunks, crcs, crcs, n_bad, ff.FF_RESTORE_SKIP_BAD)
    torch.cuda.synchronize()
    want = src.clone()
    want[3 * chunk // 2:4 * chunk // 2] = 0
    assert int(n_bad.item()) == 1 and np.array_equal(np.flatnonzero(_u32(crcs)), [3])
    assert torch.equal(t.view(torch.int16), want.view(torch.int16))


# a restore of small tensors takes longer runs of the XCDs' order above 384 MiB, and goes through the caches above 896 MiB
@pytest.mark.parametrize("nbytes", [(384 << 20) - 4096, (384 << 20) + 4096, (896 << 20) - 4096, (896 << 20) + 4096])
def test_restore_of_small_tensors_on_both_sides_of_384_mib(nbytes):
    arena = torch.empty(nbytes + (64 << 20), dtype=torch.uint8, device=DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(nbytes % 1000003)
    arena.view(torch.int64).random_(generator=gen)
    half, segs, at, left, k = arena.view(torch.bfloat16), [], 0, nbytes // 2, 0
    while left:  # 2.4 to 6.9 KB, off every line
        n = min(left, 1201 + 37 * (k % 61))
        segs.append(half[at:at + n])
        at, left, k = at + n + 1 + k % 5, left - n, k + 1
    plan = ff.ff_snapshot_plan(segs, 1 << 20)
    chunks, crcs, bad, n_bad = ff.alloc_outputs(plan, DEV)
    ff.ff_pack(plan, chunks, crcs)
    want, gaps = arena.clone(), torch.ones_like(half, dtype=torch.bool)
    for t in segs:
        gaps[(t.data_ptr() - half.data_ptr()) // 2:][:t.numel()] = False
        t.zero_()
    half.view(torch.int16)[gaps] ^= 0x55
    want.view(torch.int16)[gaps] ^= 0x55
    for flags in (0, ff.FF_RESTORE_SKIP_BAD):
        ff.ff_restore(plan, chunks, crcs, bad, n_bad, flags)
        torch.cuda.synchronize()
        assert int(n_bad.item()) == 0 and torch.equal(arena, want)
        half[~gaps] = 0
