"""SSIM in strips of columns (many pixels) against SSIM in tiles (few): the
same views in one batch, which takes the strips, and one by one, which takes
the tiles.  Widths around the strip's own 236 columns and heights around its
rows, one-pixel views, both masks.

Every loss term and gradient is a mean over its own view, so a view of a batch
has the values it has alone, up to float32 rounding.  A window's variance is a
difference of sums near 1 (rounded at 2^-24, about ten times) added to 9e-4, so
single derivatives are off by up to 10 2^-24 / 9e-4 = 7e-4 and the norm over a
view, whose variances are mostly far larger, by some 1e-6: TOL, 2e-5 of the
gradient's norm, leaves room for flat views; 1e-4 relative for the SSIM term.
Between the two paths twice that.
Pixels that are not finite spoil the same gradients in both: those within two
windows of them.
"""
import ctypes

import numpy as np
import pytest

import oracle
from paper_2603_27781_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 2e-5
SIZES = [(236, 24), (237, 25), (472, 41), (473, 40), (1, 1), (3, 200), (235, 7), (700, 23), (256, 72), (1200, 73),
         (246, 96), (64, 3)]


def _opts(use_obs):
    from paper_2603_27781_amd import _lib
    o = _lib.GsSlamLossOpts()
    _lib.load().gs_default_slam_loss_opts(ctypes.byref(o))
    o.ssim_lambda, o.w_sem = 0.2, 0.0
    o.flags = _lib.GS_LOSS_OBS_MASK if use_obs else 0
    return o


def _loss(sizes, out, rgb, dep, o):
    from paper_2603_27781_amd import raster
    views = [wl.make_view(W, H, 0.8 * max(W, H), np.eye(4)) for (W, H) in sizes]
    cfg = raster.Config()
    r = raster.Rasterizer(1, 0, raster.Views(views, cfg.tile), cfg, capacity=1024)
    r.slam_loss(*(torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (rgb, dep)), None, None, o,
                out=torch.from_numpy(np.ascontiguousarray(out)).cuda())
    torch.cuda.synchronize()
    return r.grad_out.cpu().numpy(), r.slam_terms.cpu().numpy()


TALL = [(473, 145), (237, 73), (1, 1)]


def _images(sizes):
    rng = np.random.default_rng(5)
    li = wl.loss_images(rng, sizes, 0, 0)
    return sizes, li.out, li.rgb_t, li.depth_t


@pytest.mark.parametrize("use_obs", [False, True])
@pytest.mark.parametrize("sizes", [SIZES * 4, TALL * 18, [(1200, 680)] * 8], ids=["40", "56", "72"])  # rows of a strip
def test_strips_against_tiles(sizes, use_obs):
    sizes, out, rgb, dep = _images(sizes)
    o = _opts(use_obs)
    g, terms = _loss(sizes, out, rgb, dep, o)
    total, off = 0.0, 0
    for W, H in sizes:
        sl = slice(off, off + W * H)
        ga, ta = _loss([(W, H)], out[:, sl], rgb[:, sl], dep[sl], o)
        scale = np.linalg.norm(ga[:3].astype(np.float64))
        assert np.linalg.norm(g[:3, sl].astype(np.float64) - ga[:3]) <= 2 * TOL * scale, (W, H)
        total += ta[1]
        off += W * H
    assert terms[1] == pytest.approx(total, rel=2e-4)


def test_strips_against_oracle():
    sizes, out, rgb, dep = _images(SIZES * 4)
    o = _opts(False)
    g, terms = _loss(sizes, out, rgb, dep, o)
    oo = oracle.SlamLossOpts(w_color=o.w_color, w_depth=o.w_depth, w_sem=0.0, ssim_lambda=o.ssim_lambda,
                             tau_obs=o.tau_obs, tau_unobs=o.tau_unobs, obs_factor=o.obs_factor,
                             unobs_factor=o.unobs_factor, use_obs=False)
    gref, tref = oracle.slam_loss(out, sizes, rgb, dep, None, None, oo)[:2]
    assert np.linalg.norm(g[:3] - gref[:3]) <= TOL * np.linalg.norm(gref[:3])
    assert terms[1] == pytest.approx(tref[1], rel=1e-4)


@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_not_finite(value):
    sizes, out, rgb, dep = _images(SIZES * 4)
    o = _opts(False)
    off = sum(W * H for W, H in sizes[:9])  # the 1200x73 view
    W, H = sizes[9]
    out[1, off + 36 * W + 500] = value
    rgb[2, off + 2 * W + 237] = value
    g, _ = _loss(sizes, out, rgb, dep, o)
    sl = slice(off, off + W * H)
    ga, _ = _loss([(W, H)], out[:, sl], rgb[:, sl], dep[sl], o)
    fin = np.isfinite(ga[:3])
    assert not fin.all()
    assert np.array_equal(np.isfinite(g[:3, sl]), fin)
    assert np.isfinite(g[:3, :off]).all() and np.isfinite(g[:3, off + W * H:]).all()
    d = np.where(fin, g[:3, sl].astype(np.float64) - np.where(fin, ga[:3], 0.0), 0.0)
    assert np.linalg.norm(d) <= 2 * TOL * np.linalg.norm(ga[:3][fin].astype(np.float64))


# wide and tall enough for strips of 24, 40, 56 and 72 rows once, three, six
# and four times: whole strips and one column more or less, short last strips
WIDE = [(944, 243), (943, 241), (1180, 145), (236, 96), (237, 73), (1, 1), (3, 20), (700, 23), (708, 71)]


@pytest.mark.parametrize("use_obs", [False, True])
@pytest.mark.parametrize("times", [1, 3, 6, 4])
def test_strips_of_each_height_against_tiles(times, use_obs):
    test_strips_against_tiles(WIDE * times, use_obs)


def test_wide_strips_against_oracle():
    sizes, out, rgb, dep = _images(WIDE * 3)
    o = _opts(False)
    g, terms = _loss(sizes, out, rgb, dep, o)
    oo = oracle.SlamLossOpts(w_color=o.w_color, w_depth=o.w_depth, w_sem=0.0, ssim_lambda=o.ssim_lambda,
                             tau_obs=o.tau_obs, tau_unobs=o.tau_unobs, obs_factor=o.obs_factor,
                             unobs_factor=o.unobs_factor, use_obs=False)
    gref, tref = oracle.slam_loss(out, sizes, rgb, dep, None, None, oo)[:2]
    assert np.linalg.norm(g[:3] - gref[:3]) <= TOL * np.linalg.norm(gref[:3])
    assert terms[1] == pytest.approx(tref[1], rel=1e-4)


@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("times", [1, 3, 6, 4])
def test_not_finite_in_wide_strips(value, times):
    sizes, out, rgb, dep = _images(WIDE * times)
    o = _opts(False)
    off = sum(W * H for W, H in sizes[:2])  # the 1180x145 view
    W, H = sizes[2]
    out[1, off + 71 * W + 500] = value
    rgb[2, off + 2 * W + 237] = value
    out[0, off + 140 * W + 705] = -value
    g, _ = _loss(sizes, out, rgb, dep, o)
    sl = slice(off, off + W * H)
    ga, _ = _loss([(W, H)], out[:, sl], rgb[:, sl], dep[sl], o)
    fin = np.isfinite(ga[:3])
    assert not fin.all()
    assert np.array_equal(np.isfinite(g[:3, sl]), fin)
    assert np.isfinite(g[:3, :off]).all() and np.isfinite(g[:3, off + W * H:]).all()
    d = np.where(fin, g[:3, sl].astype(np.float64) - np.where(fin, ga[:3], 0.0), 0.0)
    assert np.linalg.norm(d) <= 2 * TOL * np.linalg.norm(ga[:3][fin].astype(np.float64))


def test_narrow_views_are_not_filtered_in_strips():
    """Eight 30x3000 views have the pixels of eight 3000x30 ones and take no
    more than twice as long (in strips, 236 columns wide, 2.4 times; in tiles
    1.5)."""
    from paper_2603_27781_amd import raster
    took = []
    for size in ((30, 3000), (3000, 30)):
        sizes = [size] * 8
        P = 8 * 90000
        views = [wl.make_view(W, H, 100.0, np.eye(4)) for W, H in sizes]
        r = raster.Rasterizer(1, 0, raster.Views(views, 16), raster.Config(), capacity=1024)
        r.out.uniform_()
        rgb, dep = torch.rand(3, P, device="cuda"), torch.rand(P, device="cuda")
        o = _opts(True)
        best = 1e9
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                r.slam_loss(rgb, dep, None, None, o)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) / 10)
        took.append(best)
    print(took)
    assert took[0] <= 2 * took[1]
