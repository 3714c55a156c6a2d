"""The masks' median and the loss sums at the sizes where their kernels
change: blocks of 4096 pixels, residuals that share or split the digits of
the radix select, views without a valid depth, and pixel counts on both
sides of the one-launch sum (8192 partials of 256 pixels)."""
import numpy as np
import pytest

import oracle
from paper_2603_27781_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _slam(sizes, depth, depth_t, rgb=None, rgb_t=None):
    from paper_2603_27781_amd import raster
    P = sum(w * h for w, h in sizes)
    views = [wl.make_view(w, h, 50.0, np.eye(4)) for w, h in sizes]
    r = raster.Rasterizer(1, 0, raster.Views(views, 16), raster.Config(), capacity=64)
    out = np.zeros((5, P), np.float32)
    out[3], out[4] = depth, 1.0
    if rgb is not None:
        out[:3] = rgb
    r.out.copy_(torch.from_numpy(out))
    t = torch.from_numpy(np.zeros((3, P), np.float32) if rgb_t is None else rgb_t).cuda()
    for _ in range(2):  # the second call on a workspace that holds the first one's counts
        r.slam_loss(t, torch.from_numpy(depth_t).cuda())
    torch.cuda.synchronize()
    return r


def _residuals(kind, n, rng):
    if kind == "equal":
        return np.full(n, 0.25, np.float32)
    if kind == "low bits":  # one top digit, every low one
        return (np.uint32(0x3E800000) + rng.integers(0, 1 << 10, n, dtype=np.uint32)).view(np.float32)
    if kind == "middle bits":
        return (np.uint32(0x3E800000) + (rng.integers(0, 1 << 10, n, dtype=np.uint32) << 10)).view(np.float32)
    if kind == "wide":
        return np.exp(rng.uniform(-60, 60, n)).astype(np.float32)
    r = rng.uniform(0, 1, n).astype(np.float32)
    r[rng.random(n) < 0.6] = np.inf if kind == "inf" else np.nan
    return r


@pytest.mark.parametrize("kind", ["equal", "low bits", "middle bits", "wide", "inf", "nan"])
@pytest.mark.parametrize("sizes", [[(1, 1)], [(2, 1), (1, 3)], [(4095, 1)], [(64, 64)], [(4097, 1), (90, 91), (5, 1)]],
                         ids=lambda s: "+".join("%dx%d" % p for p in s))
def test_median_is_exact(sizes, kind):
    rng = np.random.default_rng(len(kind) + len(sizes))
    P = sum(w * h for w, h in sizes)
    # D* = 2^-100: D - D* rounds to D, so the residuals are D's bits
    dt = np.full(P, 2.0 ** -100, np.float32)
    d = _residuals(kind, P, rng)
    off = 0
    for k, (w, h) in enumerate(sizes):  # some depths missing; all of the second view's
        s = slice(off, off + w * h)
        dt[s][rng.random(w * h) < (1.0 if k == 1 else 0.1)] = 0.0
        off += w * h
    r = _slam(sizes, d, dt)
    got, off = r.median.cpu().numpy(), 0
    for k, (w, h) in enumerate(sizes):
        s = slice(off, off + w * h)
        want = np.float32(oracle.depth_median(d[s], dt[s]))
        assert got[k].view(np.uint32) == want.view(np.uint32) or (np.isnan(got[k]) and np.isnan(want)), (k, got, want)
        off += w * h


@pytest.mark.parametrize("h", [8191, 8192, 8193, 16400])
def test_loss_sums_at_the_one_launch_limit(h):
    """256 pixels per partial.  The terms are FP64 sums of binary32 terms:
    1e-12 relative against numpy's."""
    rng = np.random.default_rng(h)
    P = 256 * h
    d, dt = rng.uniform(1, 2, P).astype(np.float32), rng.uniform(1, 2, P).astype(np.float32)
    rgb, rgb_t = rng.random((3, P)).astype(np.float32), rng.random((3, P)).astype(np.float32)
    r = _slam([(256, h)], d, dt, rgb, rgb_t)
    terms = r.slam_terms.cpu().numpy()
    depth = np.abs(d - dt).astype(np.float64).sum() / P
    # (1 - lambda) w / (3 P) is rounded to binary32 once
    gc = float((np.float32(1.0) - np.float32(0.2)) * np.float32(0.5) / (np.float32(3.0) * np.float32(P)))
    colour = np.abs(rgb - rgb_t).astype(np.float64).sum() * gc
    assert abs(terms[2] - depth) <= 1e-12 * depth
    assert abs(terms[0] - colour) <= 1e-12 * colour
    assert abs(terms[4] - terms[:4].sum()) <= 1e-12 * terms[4]
