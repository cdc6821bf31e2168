"""The optimizer step's sub-blocks of 512 elements (8 KiB of a RAW segment) at the sizes where they
can go wrong: around a lane's slot, a row, a sub-block, a workgroup's eight of them and a block, with chunk boundaries that cut blocks anywhere, and on
tensors that start off every alignment."""
import numpy as np
import pytest
import torch

from paper_2512_03644_amd import binding as ff
from paper_2512_03644_amd import workloads as wl
from test_gpu_parity import DEV, HP, _adam_and_compare, _chained_and_compare

pytestmark = pytest.mark.gpu

SHORT_STEP = 80 << 20  # a step over a larger buffer has kernels of its own
EDGES = [1, 2, 3, 4, 5, 7, 8, 9, 255, 256, 257, 259, 511, 512, 513, 1023, 1024, 1025, 1027, 3583, 3584, 3585,
         4095, 4096, 4097, 8188, 8191, 8192, 8193, 8197, 16384 + 1022]


def _raw(numels, dtype, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return [torch.randn(n, device=DEV, generator=g).to(dtype) for n in numels]


@pytest.mark.parametrize("chunk", [1024, 2048, 1 << 15, 1 << 22])
def test_block_edges_in_place_and_chained(oracle, chunk):
    raw = _raw([1, 3, 7, 8, 9, 511, 4095, 4096, 4097, 16383, 16384, 16385 + 4096], torch.bfloat16, chunk)
    extra = [(5 * i, t) for i, t in enumerate(raw)]
    _adam_and_compare(oracle, EDGES, chunk, seed=chunk, hp=dict(HP, step=3), extra_raw=extra)
    _chained_and_compare(oracle, EDGES, chunk, seed=chunk + 1, steps=2, half=torch.float16,
                         loss_scale=1024.0, extra_raw=extra)


# of a short step, of a long one with a tally, and of one without
@pytest.mark.parametrize("half", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("chunk,largest", [(1 << 15, 3300001), (1 << 17, 3300001), (1 << 22, 3300001), (1 << 15, 6000001),
                                           (1 << 22, 6000001), (1 << 17, 10500001)])
def test_results_through_the_image(oracle, chunk, largest, half):
    # a launch of more than 768 workgroups whose streams lie off the lines: whole workgroups store through LDS,
    # at every edge and behind every cut
    numels = EDGES + [largest, 4096 * 3 + 512, 150001]
    assert (14 * sum(numels) > SHORT_STEP) == (largest > 3300001)
    assert (sum(numels) > 2560 * 4096) == (largest > 6000001)
    _adam_and_compare(oracle, numels, chunk, seed=chunk + 3,
                      hp=dict(HP, step=3), half=half, loss_scale=1024.0 if half == torch.float16 else 1.0)


@pytest.mark.parametrize("n", [3, 6])
def test_results_of_a_long_launch_on_the_lines(oracle, n):
    numels = [1 << 20] * n + [262144]
    assert (14 * sum(numels) > SHORT_STEP) == (n == 6)
    _adam_and_compare(oracle, numels, 1 << 20, seed=31, hp=dict(HP, step=2))


@pytest.mark.parametrize("chunk", [1024, 1 << 14, 1 << 20])
def test_many_raw_tensors_in_a_chunk(oracle, chunk):
    # workgroups whose wavefronts are at many RAW tensors of one chunk, or of two, some behind a parameter
    sizes = torch.randint(1, 3000, (300,), generator=torch.Generator().manual_seed(chunk)).tolist()
    raw = _raw(sizes + [1] * 40 + [20000], torch.bfloat16, chunk)
    extra = [(12 if i >= 30 else 5, t) for i, t in enumerate(raw)]
    _adam_and_compare(oracle, [700, 5, 9000], chunk, seed=chunk, hp=dict(HP, step=2), extra_raw=extra)
    _chained_and_compare(oracle, [700, 5, 9000], chunk, seed=chunk, steps=2, extra_raw=extra)


@pytest.mark.parametrize("shift", [1, 3, 7])
def test_step_on_tensors_off_every_alignment(shift):
    """Tensors and gradients that start `shift` elements into an allocation give the same snapshot,
    CRCs and state as aligned ones."""
    numels, chunk = [5, 1030, 8192, 20001], 1 << 14
    a = wl.param_shard("a", numels, chunk, 5 + shift, DEV, with_grads=True)

    def moved(t):
        room = torch.zeros(t.numel() + shift + 8, dtype=t.dtype, device=DEV)
        room[shift:shift + t.numel()] = t
        return room[shift:shift + t.numel()], room

    b, rooms = [], []
    for t in a.segments + [p.grad for p in a.params]:
        view, room = moved(t)
        b.append(view)
        rooms.append((room, t.numel()))
    segs_b, grads_b = b[:len(a.segments)], b[len(a.segments):]
    kinds = [ff.FF_KIND_W16, ff.FF_KIND_MASTER, ff.FF_KIND_M, ff.FF_KIND_V] * len(numels)
    pids = [k for k in range(len(numels)) for _ in range(4)]
    got = []
    for segs, grads in ((a.segments, [p.grad for p in a.params]), (segs_b, grads_b)):
        plan = ff.ff_snapshot_plan(segs, chunk, 0, kinds, pids)
        chunks, crcs, _, _ = ff.alloc_outputs(plan, DEV)
        ff.ff_adam_step_snapshot(plan, grads, HP, chunks, crcs)
        torch.cuda.synchronize()
        got.append((chunks, crcs))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    for x, y, (room, n) in zip(a.segments, segs_b, rooms):
        assert torch.equal(x, y)
        assert not room[:shift].any() and not room[shift + n:].any()  # nothing around it is touched


@pytest.mark.parametrize("high", [0, 1])
def test_every_weight_of_the_matrix_products(oracle, high):
    # With lr = 0 the master weights stay, so the streams can be chosen bit by bit: one element with one bit
    # in each sub-block of 512, so that every place of a lane's slots has every bit in every quarter of the
    # wavefront (the 16-bit weights where the bit is in the upper half), and a RAW tensor likewise.
    n = 512 * 512
    e = np.arange(512)
    master = np.zeros((512, 512), np.uint32)
    master[e, e] = np.uint32(1) << (16 * high + e // 4 % 16).astype(np.uint32)
    raw = np.zeros((2048, 2048), np.uint32)                    # sub-blocks of 8 KiB
    d = np.arange(2048)
    raw[d, d] = np.uint32(1) << (16 * high + d // 4 % 16).astype(np.uint32)

    def f32(a):
        return torch.from_numpy(a.reshape(-1).view(np.float32)).to(DEV)

    p, m, v, x = f32(master), torch.zeros(n, device=DEV), torch.zeros(n, device=DEV), f32(raw)
    w = torch.zeros(n, dtype=torch.bfloat16, device=DEV)
    chunk = 1 << 20
    plan = ff.ff_snapshot_plan([x, w, p, m, v], chunk, 0,
                               [ff.FF_KIND_RAW, ff.FF_KIND_W16, ff.FF_KIND_MASTER, ff.FF_KIND_M, ff.FF_KIND_V],
                               [0] * 5)
    chunks, crcs, _, _ = ff.alloc_outputs(plan, DEV)
    ff.ff_adam_step_snapshot(plan, [torch.zeros_like(w)], dict(HP, lr=0.0, weight_decay=0.0, step=1), chunks, crcs)
    torch.cuda.synchronize()
    got = chunks.cpu().numpy()
    half = torch.from_numpy(master.reshape(-1).view(np.float32)).to(torch.bfloat16).view(torch.int16).numpy()
    want = np.concatenate([raw.reshape(-1).view(np.uint8), half.view(np.uint8), master.reshape(-1).view(np.uint8),
                           np.zeros(8 * n, np.uint8)])
    assert np.array_equal(got[:want.size], want) and not got[want.size:].any()
    want_crcs = [oracle.crc32c(got[k:k + chunk]) for k in range(0, got.size, chunk)]
    assert np.array_equal(crcs.cpu().numpy().view(np.uint32), np.array(want_crcs, np.uint32))


# one room for the gradient pointers, the next, a launch's end and a second launch
@pytest.mark.parametrize("n", [64, 65, 384, 385, 2047, 2048, 2049, 4100])
def test_so_many_groups(oracle, n):
    numels = torch.randint(1, 40, (n,), generator=torch.Generator().manual_seed(n)).tolist()
    _adam_and_compare(oracle, numels, 1 << 14, seed=n)
    _chained_and_compare(oracle, numels, 1 << 14, seed=n + 1, steps=2)


# long chained steps that know no tally have kernels of their own: every edge, with RAW tensors between and more groups than one
# launch takes; and the same of a short step
@pytest.mark.parametrize("times", [67, 70])
@pytest.mark.parametrize("half", [torch.bfloat16, torch.float16])
def test_block_edges_of_long_chained_steps(oracle, half, times):
    numels = EDGES * times
    assert len(numels) > 2048 and (14 * sum(numels) > SHORT_STEP) == (times == 70)
    extra = [(5 * i, t) for i, t in enumerate(_raw([1, 7, 511, 4096, 16385 + 4096], torch.bfloat16, times))] if times == 70 else None
    _chained_and_compare(oracle, numels, 1 << 15, seed=67, steps=2, half=half,
                         loss_scale=1024.0 if half == torch.float16 else 1.0, extra_raw=extra)


# steps over more than 80 MiB have kernels of their own: every edge in place, behind cuts without a tally and, with one, in one
# chunk; and cuts in a short step
@pytest.mark.parametrize("times,chunk", [(55, 1 << 15), (69, 1 << 15), (1, 1 << 27)])
@pytest.mark.parametrize("half", [torch.bfloat16, torch.float16])
def test_block_edges_of_long_steps(oracle, times, chunk, half):
    assert (max(14 * sum(EDGES * times), chunk) > SHORT_STEP) == (times != 55) and (31 * times > 2048) == (times == 69)
    scale = 1024.0 if half == torch.float16 else 1.0
    extra = [(5 * i, t) for i, t in enumerate(_raw([1, 7, 511, 4096, 16385 + 4096], torch.bfloat16, times))]
    _adam_and_compare(oracle, EDGES * times, chunk, seed=times, hp=dict(HP, step=3), half=half, loss_scale=scale,
                      extra_raw=extra)
    if times == 1:
        _chained_and_compare(oracle, EDGES, chunk, seed=3, steps=2, half=half, loss_scale=scale, extra_raw=extra)


def test_captured_step_over_many_groups():
    # 16 KiB of kernel arguments in a graph node: every replay, with eager work between them, equals the eager step
    numels = [7 + 3 * i for i in range(500)]
    shard = wl.param_shard("a", numels, 1 << 16, 44, DEV, with_grads=True)
    plan = ff.plan_for_shard(shard)
    grads = [p.grad for p in shard.params]
    chunks, crcs, _, _ = ff.alloc_outputs(plan, DEV)

    def step():
        ff.ff_adam_step_snapshot(plan, grads, HP, chunks, crcs)

    step()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for rep in range(3):
        start = [t.clone() for t in shard.segments]
        for t in grads:
            t.mul_(0.5)
        chunks.fill_(0xA5)
        graph.replay()
        torch.cuda.synchronize()
        got = [t.clone() for t in shard.segments] + [chunks.clone(), crcs.clone()]
        for t, s0 in zip(shard.segments, start):
            t.copy_(s0)
        chunks.fill_(0xA5)
        step()
        torch.cuda.synchronize()
        for a, b in zip(got, list(shard.segments) + [chunks, crcs]):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), rep


# one launch on the default stream, two on others: chunks of one contribution, of one word of 32, of several, and of
# more than the words take (a parameter of 1221 workgroups in one chunk); a long end to clear; again and again
@pytest.mark.parametrize("chunk,numels", [(1 << 10, [100, 3]), (1 << 19, [4096 * 31 + 5]), (1 << 22, [4096 * 40 + 1, 77, 4096 * 12]),
                                          (1 << 25, [4096 * 300 + 9, 2]), (1 << 27, [5000001])])
@pytest.mark.parametrize("half", [torch.bfloat16, torch.float16])
def test_step_in_one_launch_and_in_two(chunk, numels, half):
    kinds = [ff.FF_KIND_W16, ff.FF_KIND_MASTER, ff.FF_KIND_M, ff.FF_KIND_V] * len(numels) + [ff.FF_KIND_RAW]
    pids = [k for k in range(len(numels)) for _ in range(4)] + [0]
    gen = torch.Generator(device=DEV)
    gen.manual_seed(chunk)

    def rand(n, std, dtype=torch.float32):
        return torch.randn(n, device=DEV, generator=gen).mul_(std).to(dtype)

    segs = []
    for n in numels:
        segs += [rand(n, 0.02, half), rand(n, 0.02), rand(n, 1e-3), rand(n, 1e-3).square_()]
    segs.append(rand(1001, 1.0, torch.bfloat16))
    grads = [rand(n, 1e-3, half) for n in numels]
    n_inf = 0
    if half == torch.float16:
        grads[0][::3].fill_(float("inf"))
        n_inf = (numels[0] + 2) // 3
    plan = ff.ff_snapshot_plan(segs, chunk, 0, kinds, pids)
    start, got = [t.clone() for t in segs], []
    side = torch.cuda.Stream()
    count = torch.zeros(1, dtype=torch.int64, device=DEV)
    chunks, crcs, _, _ = ff.alloc_outputs(plan, DEV)
    for stream in (None, None, side, None, side):
        for t, s0 in zip(segs, start):
            t.copy_(s0)
        chunks.fill_(0xA5)
        crcs.fill_(7)
        count.fill_(99)
        torch.cuda.synchronize()
        if half == torch.float16:
            ff.ff_adam_step_snapshot_f16(plan, grads, HP, 1.0, count, chunks, crcs, stream=stream)
        else:
            ff.ff_adam_step_snapshot(plan, grads, HP, chunks, crcs, stream=stream)
        torch.cuda.synchronize()
        if half == torch.float16:
            assert int(count.item()) == n_inf
        assert not chunks[plan.payload_bytes:].any()
        out = [chunks.clone(), crcs.clone()] + [t.clone() for t in segs]
        got = got or out
        for a, b in zip(got, out):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
