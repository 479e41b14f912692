"""GPU tests of the batched build + consecutive-pair merge and its graph:
every frame equals a standalone build and the oracle, every pair union
equals the oracle's, replays of the captured graph are bitwise identical to
the eager call, and no tuning changes a bit."""
import numpy as np
import pytest
import torch

import gen
import oracle
from helpers import dev, say, u32, u64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def frames():
    # 12 LiDAR frames of a random walk, sizes log-uniform in [64, 40k], one
    # of them emptied, so the pair merges see empty operands too
    d = gen.c4_frames(seed=77, nframes=12, size_lo=64, size_hi=40_000)
    xyz, off = d["xyz"], d["off"].copy()
    keep = np.ones(len(xyz), bool)
    keep[off[5]:off[6]] = False  # frame 5 empty
    sizes = np.diff(off)
    sizes[5] = 0
    off2 = np.zeros_like(off)
    off2[1:] = np.cumsum(sizes)
    return dict(xyz=np.ascontiguousarray(xyz[keep]), off=off2, grid=d["grid"])


def _check(gpu, frames, out):
    xyz, off, g = frames["xyz"], frames["off"], frames["grid"]
    F = len(off) - 1
    ko = out.key_off.cpu().numpy()
    keys = u64(out.keys)
    cnts = u32(out.counts)
    want = []
    for f in range(F):
        wk, wc = oracle.build(xyz[off[f]:off[f + 1]], g)
        want.append(wk)
        assert np.array_equal(keys[ko[f]:ko[f + 1]], wk), f
        assert np.array_equal(cnts[ko[f]:ko[f + 1]], wc), f
    mo, mc = out.merged_off.cpu().numpy(), out.merged_cnt.cpu().numpy()
    merged = u64(out.merged)
    for f in range(F - 1):
        wm, _ = oracle.merge(want[f], want[f + 1], g.depth, g.key_mode)
        assert mc[f] == len(wm), f
        assert np.array_equal(merged[mo[f]:mo[f] + mc[f]], wm), f


def test_batch_matches_oracle(gpu, frames):
    out = gpu.cga_batch_build_merge(dev(frames["xyz"]), dev(frames["off"]), frames["grid"])
    torch.cuda.synchronize()
    _check(gpu, frames, out)


def test_batch_frame_equals_standalone_build(gpu, frames):
    xyz, off, g = frames["xyz"], frames["off"], frames["grid"]
    out = gpu.cga_batch_build_merge(dev(xyz), dev(off), g)
    for f in (0, 3, 5, 11):
        k, c = gpu.cga_build(dev(xyz[off[f]:off[f + 1]]), g)
        assert torch.equal(out.frame(f), k), f


@pytest.mark.parametrize("tune", [(4, 8), (8, 12), (11, 16), (9, 8)])
def test_batch_tunings_identical(gpu, frames, tune):
    ref = gpu.cga_batch_build_merge(dev(frames["xyz"]), dev(frames["off"]), frames["grid"])
    out = gpu.cga_batch_build_merge(dev(frames["xyz"]), dev(frames["off"]), frames["grid"],
                                    tune=tune)
    u = int(ref.key_off[-1].item())
    assert torch.equal(ref.keys[:u], out.keys[:u]) and torch.equal(ref.key_off, out.key_off)
    assert torch.equal(ref.merged_cnt, out.merged_cnt)


def test_batch_single_and_tiny(gpu):
    g = gen.Grid((0.0, 0.0, 0.0), 1.0, 6, gen.KEY_MORTON)
    rng = np.random.default_rng(5)
    for sizes in ([0], [7], [0, 0, 3], [5000, 1, 0, 4097]):
        xyz = rng.integers(0, 64, (sum(sizes), 3)).astype(np.float32)
        off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
        out = gpu.cga_batch_build_merge(dev(xyz), dev(off), g)
        _check(gpu, dict(xyz=xyz, off=off, grid=g), out)


def test_batch_segment_tile_edges(gpu):
    """Frames of exactly one tile, one tile and one key, two tiles, with
    empty frames between, under a fixed 4096-key tile (the frame-segmented
    sort): every frame sorted within its own range."""
    g = gen.Grid((0.0, 0.0, 0.0), 1.0, 10, gen.KEY_MORTON)
    rng = np.random.default_rng(11)
    sizes = [4096, 0, 4097, 8192, 1, 0, 0, 8191, 12289, 2]
    xyz = rng.integers(0, 1024, (sum(sizes), 3)).astype(np.float32)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    for tune in ((8, 16), (7, 16), (9, 32)):
        say("segmented batch sort, tune", tune)
        out = gpu.cga_batch_build_merge(dev(xyz), dev(off), g, tune=tune)
        _check(gpu, dict(xyz=xyz, off=off, grid=g), out)


def test_batch_many_frames_composite_sort(gpu):
    """Beyond 4096 frames the batch sorts the composite keys (frame bits
    included) in one sort: 4100 frames of 0 to 40 points, and 4096 frames
    (segmented) of the same points, both against the oracle."""
    g = gen.Grid((0.0, 0.0, 0.0), 1.0, 8, gen.KEY_MORTON)
    rng = np.random.default_rng(12)
    for nf in (4100, 4096):
        assert gpu.cga_batch_sort_bits(g, nf) == 24 + (13 if nf > 4096 else 0)
        sizes = rng.integers(0, 41, nf)
        sizes[rng.choice(nf, nf // 10, replace=False)] = 0
        xyz = rng.integers(0, 256, (int(sizes.sum()), 3)).astype(np.float32)
        off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
        say("batch of", nf, "frames,", len(xyz), "points")
        out = gpu.cga_batch_build_merge(dev(xyz), dev(off), g)
        _check(gpu, dict(xyz=xyz, off=off, grid=g), out)


@pytest.mark.parametrize("depth,nf", [(21, 2), (20, 16), (19, 128), (16, 65536)])
def test_batch_frame_bits_end_at_64(gpu, depth, nf):
    """As many frames as the composite key has room for: the last frame's end
    (key_off[F]) is the number of keys, so every pair's length is right."""
    rng = np.random.default_rng(depth)
    sizes = rng.integers(0, 3, nf) if nf > 1000 else rng.integers(1, 3000, nf)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    p = rng.uniform(0, 1, (int(off[-1]), 3)).astype(np.float32)
    p[-1] = 1.0  # the largest key in the last frame: all 64 bits set
    g = gen.Grid((0.0, 0.0, 0.0), 2.0 ** depth, depth, gen.KEY_MORTON)
    say("batch of", nf, "frames at depth", depth)
    for tune in (None, (8, 16)):
        out = gpu.cga_batch_build_merge(dev(p), dev(off), g, tune=tune)
        ko = out.key_off.cpu().numpy()
        mo, mc = out.merged_off.cpu().numpy(), out.merged_cnt.cpu().numpy()
        keys, merged = u64(out.keys), u64(out.merged)
        assert (np.diff(ko) >= 0).all() and ko[-1] <= len(p)
        for f in range(nf - 1) if nf < 1000 else (0, 1, nf // 2, nf - 3, nf - 2):
            want = [oracle.build(p[off[i]:off[i + 1]], g)[0] for i in (f, f + 1)]
            for i in (0, 1):
                assert np.array_equal(keys[ko[f + i]:ko[f + i + 1]], want[i]), f
            wm, _ = oracle.merge(want[0], want[1], g.depth, g.key_mode)
            assert mc[f] == len(wm) and np.array_equal(merged[mo[f]:mo[f] + mc[f]], wm), f


@pytest.mark.parametrize("kind", ["uniform", "same", "few", "far"])
@pytest.mark.parametrize("depth,mode", [(9, gen.KEY_MORTON), (10, gen.KEY_LINEAR),
                                        (12, gen.KEY_MORTON), (20, gen.KEY_LINEAR)])
def test_batch_buckets(gpu, depth, mode, kind):
    """Frames built by buckets (2^17 points or more on average): empty
    frames at either end and inside, one point, one bucket and one point more,
    frames over several blocks; against the oracle, and replayed as a graph."""
    g = gen.Grid((0.0, 0.0, 0.0), 2.0 ** depth, depth, mode)
    rng = np.random.default_rng(depth)
    sizes = [0, 1, 8191, 8192, 0, 30_000, 1_200_001, 4096, 70_003, 0]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    n = int(off[-1])
    p = rng.uniform(0, 1, (n, 3)).astype(np.float32)
    if kind == "same":
        p[:] = 0.3
    elif kind == "few":
        p = p[rng.integers(0, 37, n)]
    elif kind == "far":
        p *= np.float32(2.0 ** -5)
        p[::3] = 1 - p[::3]
    say("batch by buckets", depth, kind)
    xyz, doff = dev(p), dev(off)
    out = gpu.cga_batch_build_merge(xyz, doff, g)
    _check(gpu, dict(xyz=p, off=off, grid=g), out)
    u = int(out.key_off[-1].item())
    graph = gpu.BatchGraph(xyz, doff, g)
    for _ in range(2):
        graph.out.keys.fill_(0)
        graph.launch()
        torch.cuda.synchronize()
        assert graph.status() == 0
        assert torch.equal(graph.out.keys[:u], out.keys[:u])
        assert torch.equal(graph.out.counts[:u], out.counts[:u])
        assert torch.equal(graph.out.key_off, out.key_off)
        assert torch.equal(graph.out.merged_cnt, out.merged_cnt)
    graph.close()


@pytest.mark.parametrize("depth,sizes,buckets", [
    (12, [3_000_000, 20_000], True),            # above 2^21: fewer than eight samples a bucket
    (12, [150_000, 9_000_000, 150_000], True),  # one large frame among small ones: 2197 buckets
    (10, [100_000, 17_500_000, 0, 60_000, 40_000], True),  # more than 4096 points to each of 4096
    (14, [600_000], True),                      # few points, wide spans: 1171 points a bucket
    (12, [1 << 22], True), (12, [(1 << 22) + 1], False),      # the rule's ends
    (15, [3 << 20], True), (15, [(3 << 20) + 1], False),
    (12, [1 << 17] * 3 + [(1 << 17) + 1], True), (12, [1 << 17] * 3 + [(1 << 17) - 1], False)])
def test_batch_bucket_frames(gpu, depth, sizes, buckets):
    """Which batches go by buckets, and every frame against its own build by the
    radix sort."""
    rng = torch.Generator(device="cuda").manual_seed(depth)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    n = int(off[-1])
    p = torch.rand((n, 3), generator=rng, device="cuda")
    p[::2, 2] = 0.25 + 0.5 * p[::2, 0] * p[::2, 1]  # half of them on a surface
    g = gen.Grid((0.0, 0.0, 0.0), 2.0 ** depth, depth, gen.KEY_MORTON)
    say("batch of", sizes[:3], "at depth", depth)
    gpu.cga_prof_enable(["bucket_sort", "onesweep"])
    gpu.cga_prof_reset()
    try:
        out = gpu.cga_batch_build_merge(p, dev(off), g)
        torch.cuda.synchronize()
        assert (gpu.cga_prof_read("bucket_sort")[1] > 0) == buckets
        assert (gpu.cga_prof_read("onesweep")[1] > 0) == (not buckets)
    finally:
        gpu.cga_prof_disable()
        gpu.cga_prof_reset()
    ko, frames = out.key_off.cpu().tolist(), []
    for f, m in enumerate(sizes):
        k, c = gpu.cga_build(p[off[f]:off[f + 1]].contiguous(), g, tune=(8, 16))
        assert torch.equal(out.keys[ko[f]:ko[f + 1]], k), f
        assert torch.equal(out.counts[ko[f]:ko[f + 1]], c), f
        frames.append(k.clone())
    for f in range(len(sizes) - 1):
        assert torch.equal(out.pair(f), gpu.cga_merge(frames[f], frames[f + 1], g)[0]), f


def test_graph_replays_match_eager(gpu, frames):
    xyz, off, g = dev(frames["xyz"]), dev(frames["off"]), frames["grid"]
    ref = gpu.cga_batch_build_merge(xyz, off, g)
    torch.cuda.synchronize()
    u = int(ref.key_off[-1].item())
    graph = gpu.BatchGraph(xyz, off, g)
    for rep in range(3):
        # unrelated eager work between replays
        gpu.cga_build(xyz[:1000], g)
        graph.out.keys.fill_(0)
        graph.out.merged_cnt.fill_(-1)
        graph.launch()
        torch.cuda.synchronize()
        assert graph.status() == 0
        assert torch.equal(graph.out.key_off, ref.key_off), rep
        assert torch.equal(graph.out.keys[:u], ref.keys[:u]), rep
        assert torch.equal(graph.out.merged_cnt, ref.merged_cnt), rep
        assert torch.equal(graph.out.merged_off, ref.merged_off), rep
        # each pair's region holds merged_cnt keys; the rest of it is unused
        for f in range(len(ref.merged_cnt)):
            assert torch.equal(graph.out.pair(f), ref.pair(f)), (rep, f)
    graph.close()


def test_autotuner_choice_is_used_and_exact(gpu, frames):
    g = frames["grid"]
    rb, items, ms = gpu.cga_autotune_sort(key_bytes=8, key_bits=3 * g.depth, n=len(frames["xyz"]))
    say("autotune", rb, items, ms)
    assert 4 <= rb <= 11 and items in (8, 12, 16, 24, 32) and ms > 0
    k, c = gpu.cga_build(dev(frames["xyz"]), g)  # picks the recorded choice
    wk, wc = oracle.build(frames["xyz"], g)
    assert np.array_equal(u64(k), wk) and np.array_equal(u32(c), wc)


def test_autotuner_keeps_the_buckets(gpu):
    """A recorded sort is for calls that sort: builds and batches that go by
    buckets still do, and one that names a sort gets it."""
    g = gen.Grid((0.0, 0.0, 0.0), 2.0 ** 12, 12, gen.KEY_MORTON)
    n = 600_000
    gpu.cga_autotune_sort(key_bytes=8, key_bits=36, n=n)
    p = torch.rand((n, 3), generator=torch.Generator(device="cuda").manual_seed(7), device="cuda")
    off = dev(np.array([0, 250_000, n], np.int64))
    outs = []
    for tune, call in ((None, lambda t: gpu.cga_build(p, g, tune=t)),
                       ((8, 16), lambda t: gpu.cga_build(p, g, tune=t)),
                       (None, lambda t: gpu.cga_batch_build_merge(p, off, g, tune=t)),
                       ((8, 16), lambda t: gpu.cga_batch_build_merge(p, off, g, tune=t))):
        gpu.cga_prof_enable(["bucket_sort", "onesweep"])
        gpu.cga_prof_reset()
        try:
            outs.append(call(tune))
            torch.cuda.synchronize()
            launches = [gpu.cga_prof_read(x)[1] > 0 for x in ("bucket_sort", "onesweep")]
        finally:
            gpu.cga_prof_disable()
            gpu.cga_prof_reset()
        assert launches == [tune is None, tune is not None], tune
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
    u = int(outs[2].key_off[-1])
    assert torch.equal(outs[2].key_off, outs[3].key_off)
    assert torch.equal(outs[2].keys[:u], outs[3].keys[:u])
