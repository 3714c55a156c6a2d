"""Binning, bit for bit against the oracle, where its kernels change their
way: list lengths around the limits of the per-tile sort (one wavefront up to
512 keys, one workgroup up to 4096, parts that are merged beyond), chunk
counts on both sides of the look-back, chunks of 1024, 4096 and 16384 pairs
and several passes, tiles counted in more than one window, a table that does
not fit and falls back to larger chunks, 32-bit counters or the tile ranges,
a capacity that cuts the lists, and replays of a captured call."""
import numpy as np
import pytest

import oracle
from gpu_common import oracle_cfg
from paper_2603_27781_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _views(sizes, f=0.8, seed=0):
    rng = np.random.default_rng(seed)
    return [wl.make_view(w, h, f * max(w, h), wl.se3_exp(wl._random_twist(rng, 0.03, 0.03))) for w, h in sizes]


def _scene(n, seed, log_scale=-3.5, spread=1.0):
    sc = wl.box_scene(np.random.default_rng(seed), n, (-spread, -0.6 * spread, 1.5), (spread, 0.6 * spread, 4), log_scale,
                      0.4, 0)
    sc.mu[2, ::7] = sc.mu[2, 0]  # equal depths under the identity rotation: index order decides
    return sc


def _bin(sc, views, tile=16, capacity=None):
    from paper_2603_27781_amd import raster
    cfg = raster.Config(tile=tile)
    g = raster.Gaussians.from_numpy(sc)
    r = raster.Rasterizer(sc.n, 0, raster.Views(views, tile), cfg, capacity=capacity)
    if capacity is None:
        r.ensure_capacity(g)
        r.clear_trouble()
    r.project(g)
    r.bin_sort()
    return r, g, oracle.bin_instances(sc, views, oracle_cfg(cfg))


def _check(r, ref, touched):
    inst, nvis, over, gave_up = r.instance_counts()
    assert not over and not gave_up and not r.trouble()
    assert inst == ref["count"] and nvis == int((touched > 0).sum())
    assert np.array_equal(r.ranges.view(-1, 2).cpu().numpy(), ref["ranges"])
    assert np.array_equal(r.keys[:inst].cpu().numpy().view(np.uint32), ref["keys"])
    assert np.array_equal(r.sorted_gids(inst).cpu().numpy(), ref["gids"])
    first, t = r.pair_first.cpu().numpy().astype(np.int64), touched.reshape(-1).astype(np.int64)
    vis = np.nonzero(t)[0]
    assert np.array_equal(first[vis], (np.cumsum(t) - t)[vis])  # pairs in order, none skipped


@pytest.mark.parametrize("n", [1, 63, 512, 513, 1100, 4096, 4097, 9000, 20000])
def test_list_lengths(n):
    """One tile that every Gaussian reaches (and three that most reach)."""
    sc = _scene(n, n, log_scale=-1.0, spread=0.3)
    sc.mu[2] = np.maximum(sc.mu[2], 1.0)
    views = [wl.make_view(20, 20, 24.0, np.eye(4))]
    r, g, ref = _bin(sc, views)
    if n >= 512:
        assert int((ref["ranges"][:, 1] - ref["ranges"][:, 0]).max()) > 0.9 * n
    _check(r, ref, ref["dec"]["touched"])


@pytest.mark.parametrize("sizes,n,tile", [
    ([(120, 90)], 131072, 16),                              # 128 chunks: the last size by look-back
    ([(120, 90)], 131073, 16),                              # 129
    ([(200, 150)], 300001, 16),                             # 4096 pairs a chunk
    ([(64, 48), (130, 70), (17, 200)] * 4, 200003, 16),     # 16384 a chunk, uneven views
    ([(64, 48)] * 16, 1300001, 16),                         # several passes a chunk
    ([(1300, 900)], 3000, 8),                               # 18,419 tiles in one window
    ([(1500, 1500)], 3000, 8),                              # 35,344 tiles: two windows
    ([(1, 1), (9, 8), (8, 9)], 700, 8),
], ids=lambda x: str(x) if not isinstance(x, list) else "x".join(map(str, x[0])) + "*%d" % len(x))
def test_chunks_and_windows(sizes, n, tile):
    r, g, ref = _bin(_scene(n, 5), _views(sizes), tile)
    _check(r, ref, ref["dec"]["touched"])


@pytest.mark.parametrize("side,n", [(5000, 200000), (8200, 30000)], ids=["32-bit counters", "table in the ranges"])
def test_more_tiles_than_the_table_holds(side, n):
    r, g, ref = _bin(_scene(n, 6, log_scale=-5.0), [wl.make_view(side, side, 0.8 * side, np.eye(4))], 8)
    _check(r, ref, ref["dec"]["touched"])


def test_truncated_lists_hold_the_first_instances():
    sc, views = _scene(5000, 7), _views([(160, 120)])
    full, _, ref = _bin(sc, views)
    cap = ref["count"] // 2 + 7
    r, _, _ = _bin(sc, views, capacity=cap)
    inst, _, over, _ = r.instance_counts()
    assert inst == ref["count"] and over and r.trouble()
    keys, e = full.keys[:inst].cpu().numpy(), full.inst[:inst].cpu().numpy()
    keep = e < cap
    assert np.array_equal(r.inst[:cap].cpu().numpy(), e[keep])
    assert np.array_equal(r.keys[:cap].cpu().numpy(), keys[keep])
    n = r.ranges.view(-1, 2).cpu().numpy()
    assert np.array_equal(n[:, 1] - n[:, 0], np.bincount(keys[keep], minlength=len(n)))


def test_replays_of_a_captured_call_follow_the_scene():
    sc, views = _scene(9000, 8, log_scale=-2.0), _views([(90, 70), (40, 60)])
    r, g, ref = _bin(sc, views, capacity=2_000_000)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        r.project(g)
        r.bin_sort()
    for k in range(3):
        sc.mu[2] += 0.2 * k
        g.mu.copy_(torch.from_numpy(sc.mu))
        graph.replay()
        ref = oracle.bin_instances(sc, views, oracle_cfg(r.cfg))
        _check(r, ref, ref["dec"]["touched"])
        torch.ones(1000, device="cuda").sum().item()  # eager work between the replays


@pytest.mark.parametrize("sizes,n,tile,cap", [
    ([(2048, 1024)], 3000, 8, None),                             # 32,768 tiles: the last size counted in LDS
    ([(2056, 1024)], 3000, 8, None),                             # 32,896: in memory
    ([(2056, 1024)], 140000, 8, None),                           # the same without the look-back
    ([(70, 50), (2600, 900), (33, 90)], 9000, 8, None),          # one such view among small ones
    ([(2056, 1024), (40, 40)], 20000, 8, 50001),                 # capacity below the instances
    ([(8200, 8200)], 140000, 8, None),                           # counters in the tile ranges, no look-back
], ids=lambda x: "x".join(map(str, x[0])) + "*%d" % len(x) if isinstance(x, list) else str(x))
def test_tiles_counted_in_memory(sizes, n, tile, cap):
    sc, views = _scene(n, 9, log_scale=-5.0 if n > 20000 else -3.5), _views(sizes)
    r, g, ref = _bin(sc, views, tile)
    _check(r, ref, ref["dec"]["touched"])
    if cap is not None:
        full, inst = r, ref["count"]
        assert inst > cap
        r, g, _ = _bin(sc, views, tile, capacity=cap)
        got, _, over, _ = r.instance_counts()
        assert got == inst and over and r.trouble()
        e = full.inst[:inst].cpu().numpy()
        assert np.array_equal(r.inst[:cap].cpu().numpy(), e[e < cap])
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    first = [x.clone() for x in (r.ranges, r.inst[:1000], r.counts)]
    with torch.cuda.graph(graph):
        r.bin_sort()
    for _ in range(2):  # the counters are cleared by every call
        graph.replay()
        assert all(torch.equal(a, b) for a, b in zip(first, (r.ranges, r.inst[:1000], r.counts)))


def _ps_per_instance(sc, views, tile):
    from paper_2603_27781_amd import raster
    g = raster.Gaussians.from_numpy(sc)
    r = raster.Rasterizer(sc.n, 0, raster.Views(views, tile), raster.Config(tile=tile))
    r.ensure_capacity(g)
    best = 1e9
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        r.bin_sort()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b))
    return 1e9 * best / r.instance_counts().instances


def test_time_per_instance_holds_for_views_of_many_tiles():
    """Binning moves the same bytes for an instance whatever the tiles: a
    3840x2160 view at tile 8 (129,600 tiles) and a 7680x4320 one at tile 16
    take no more than four times as long for each as at 32,400 tiles (walking
    the pairs again for every 32,768 tiles took 4.8 times as long for both;
    counting in memory 0.8)."""
    sc = _scene(100000, 3, log_scale=-4.0)
    took = [_ps_per_instance(sc, [wl.make_view(w, h, 0.8 * w, np.eye(4))], tile)
            for (w, h), tile in [((3840, 2160), 16), ((3840, 2160), 8), ((7680, 4320), 16)]]
    print(took)
    assert max(took[1:]) <= 4 * took[0]


def test_time_per_instance_holds_for_few_large_gaussians():
    """1000 Gaussians that reach most of a view, 3.2 M instances, take no more
    than four times as long for each as 300,000 small ones (one workgroup for
    all of them: 6.5 times, four: 2.1)."""
    views = [wl.make_view(1200, 680, 960.0, np.eye(4))]
    few, many = (_ps_per_instance(_scene(n, 4, log_scale=ls), views, 16) for n, ls in ((1000, 0.0), (300000, -5.0)))
    print(few, many)
    assert few <= 4 * many


@pytest.mark.parametrize("sizes,n,cap", [
    ([(90, 60)], 256, None), ([(90, 60)], 257, None),    # one and two chunks of 256
    ([(90, 60)], 32768, None), ([(90, 60)], 32769, None),  # the last size of such chunks, chunks of 1024
    ([(90, 60), (31, 70)], 16385, None),
    ([(1900, 1000)] * 2, 90000, 24_000_000),             # a table of 5.2 M words, which the capacity makes room for
    ([(1900, 1000)] * 2, 90000, 6_000_000),              # and too little of it: larger chunks
], ids=lambda x: "x".join(map(str, x[0])) + "*%d" % len(x) if isinstance(x, list) else str(x))
def test_small_chunks_and_table_sizes(sizes, n, cap):
    sc, views = _scene(n, 11, log_scale=-5.0 if n > 30000 else -3.5), _views(sizes)
    r, g, ref = _bin(sc, views, 16 if cap is None else 8, capacity=cap)
    _check(r, ref, ref["dec"]["touched"])


@pytest.mark.parametrize("n,sizes", [
    (8192, [(20, 20)]), (8193, [(20, 20)]),              # two parts, three (a run without a sibling)
    (12300, [(20, 20)]), (16385, [(20, 20)] * 2),        # four and five: levels of either parity
    (40000, [(20, 20), (10, 16)]), (70001, [(16, 16)]),  # ten, eighteen
    (30000, [(90, 60)]),                                 # lists of one wavefront, one workgroup and parts together
])
def test_merged_lists(n, sizes):
    sc = _scene(n, n, log_scale=-1.0 if len(sizes) > 1 or sizes[0][0] < 90 else -2.5, spread=0.3)
    sc.mu[2] = np.maximum(sc.mu[2], 1.0)
    r, g, ref = _bin(sc, [wl.make_view(w, h, 24.0, np.eye(4)) for w, h in sizes])
    assert int((ref["ranges"][:, 1] - ref["ranges"][:, 0]).max()) > 8192 * (n < 30000) * 0.9
    for _ in range(2):
        r.bin_sort()
    _check(r, ref, ref["dec"]["touched"])


def test_time_per_instance_holds_for_long_lists():
    """Lists of some 54,000 take no more than three times as long for each
    instance as lists of some 1200 (every key looked up in all other parts of
    its list: 4.5 times; merged by levels: 1.1)."""
    few = _ps_per_instance(_scene(200000, 4, log_scale=-4.0), [wl.make_view(640, 480, 512.0, np.eye(4))], 16)
    many = _ps_per_instance(_scene(1000000, 4, log_scale=-5.0), _views([(97, 61)] * 12), 16)
    print(few, many)
    assert many <= 3 * few


@pytest.mark.parametrize("size", [(8, 8), (64, 64), (512, 1024), (513, 1024), (1024, 4096), (1024, 4104)])
def test_one_entry_per_tile(size):
    """One chunk of pairs, so one table entry per tile: 1, 64, a full block of
    the scan (8192 tiles) and a column more, eight blocks and a row more."""
    sc = _scene(200, 2, log_scale=-3.0)
    r, g, ref = _bin(sc, [wl.make_view(*size, 0.8 * max(size), np.eye(4))], 8)
    _check(r, ref, ref["dec"]["touched"])


def _give_up_calls(r, monkeypatch):
    """Five calls whose waits look once and give up; the ones that did."""
    monkeypatch.setenv("SGS_LOOKBACK_SPIN", "0")
    for _ in range(5):
        r.clear_trouble()
        r.bin_sort()
        if r.instance_counts().lookback_gave_up:
            assert r.trouble()
            yield r.ranges.view(-1, 2).cpu().numpy().copy()
    monkeypatch.delenv("SGS_LOOKBACK_SPIN")


@pytest.mark.parametrize("size,tile", [((640, 480), 16), ((3840, 2160), 8)], ids=["table", "one entry per tile"])
def test_give_up_of_the_tile_scan(monkeypatch, size, tile):
    """More than 128 chunks, whose offsets need no wait: only the scan of the
    tiles (19 and 16 workgroups) can give up, and every list is left empty."""
    sc, views = _scene(140000, 12, log_scale=-5.0), _views([size])
    r, g, ref = _bin(sc, views, tile)
    gave_up = list(_give_up_calls(r, monkeypatch))
    assert gave_up, "no wait gave up in five calls with a spin limit of 0"
    assert not any(x.any() for x in gave_up)
    r.clear_trouble()
    r.bin_sort()
    _check(r, ref, ref["dec"]["touched"])


def test_give_up_of_a_merge(monkeypatch):
    """More than 128 chunks and at most 64 tiles, one workgroup of the scan:
    only the merges of lists of more than 4096 can give up, and they leave
    the list they were for empty and the others as they are."""
    sc, views = _scene(140000, 13, log_scale=-3.0, spread=0.6), [wl.make_view(90, 60, 72.0, np.eye(4))]
    r, g, ref = _bin(sc, views)
    want = ref["ranges"]
    n = want[:, 1] - want[:, 0]
    assert len(n) <= 64 and (n > 4096).any()
    seen = False
    for got in _give_up_calls(r, monkeypatch):
        empty = (got == 0).all(1)
        assert empty.any() and (empty <= (n > 4096)).all()
        assert np.array_equal(got[~empty], want[~empty])
        gids = r.sorted_gids(ref["count"]).cpu().numpy()
        for a, b in got[~empty]:
            assert np.array_equal(gids[a:b], ref["gids"][a:b])
        seen = True
    assert seen, "no wait gave up in five calls with a spin limit of 0"
    r.clear_trouble()
    r.bin_sort()
    _check(r, ref, ref["dec"]["touched"])
