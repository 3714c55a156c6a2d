"""Launch shapes the library chooses itself: the order of the tiles over the
XCDs (runs whose length follows the image) and the LDS batch of the
compositing kernels (tile, feature count, gradients).

Neither changes a pixel's arithmetic, so the forward equals the persistent
launch (which has no tile order) bit for bit, and the backward equals it up
to the order in which a tile's wavefront totals are added: binary32 sums of
at most 16 such totals, 1e-4 of the tensor's maximum (16 eps = 2e-6, times
50 for cancellation among them)."""
import dataclasses

import numpy as np
import pytest

from paper_2603_27781_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# one tile; fewer tiles than the shortest run; a last run that is nearly
# empty; 9 runs over 8 XCDs; just under and over 512 tiles of side 16 (the
# first size with a longer run); two views, the second starting inside a run
SIZES = [[(9, 5)], [(48, 16)], [(272, 240)], [(144, 64)], [(365, 349)], [(512, 256)], [(50, 33), (161, 97)]]


def _case(sizes, F, tile, seed, **kw):
    from paper_2603_27781_amd import raster
    rng = np.random.default_rng(seed)
    sc = wl.box_scene(rng, 600, (-1, -0.7, 1.5), (1, 0.7, 4), -3.2, 0.4, F)
    views = [wl.make_view(w, h, 0.8 * max(w, h), wl.se3_exp(wl._random_twist(rng, 0.05, 0.05))) for w, h in sizes]
    cfg = raster.Config(tile=tile, **kw)
    g = raster.Gaussians.from_numpy(sc)
    r = raster.Rasterizer(sc.n, F, raster.Views(views, tile), cfg)
    r.ensure_capacity(g)
    return r, g


def _run(r, g, cfg, grad_out, flags):
    r.cc = cfg.c()
    out = r.forward(g).clone()
    grads = g.zeros_like()
    r.render_bwd(g, grad_out, flags, grads)
    tw = r.pose_grad(g).clone()
    torch.cuda.synchronize()
    return out, r.T_final.clone(), r.last.clone(), grads.tensors() + [tw]


def _agree(r, g, flags):
    grad_out = torch.randn(r.out.shape, generator=torch.Generator("cuda").manual_seed(5), device="cuda")
    a = _run(r, g, r.cfg, grad_out, flags)
    b = _run(r, g, dataclasses.replace(r.cfg, persistent=1, lds_batch=64, lds_batch_bwd=64), grad_out, flags)
    for x, y in zip(a[:3], b[:3]):
        assert torch.equal(x, y)
    assert float(a[0].abs().max()) > 0
    for x, y in zip(a[3], b[3]):
        if y.numel() and float(y.abs().max()) > 0:
            assert float((x - y).abs().max()) <= 1e-4 * float(y.abs().max())
        else:
            assert torch.equal(x, y)


@pytest.mark.parametrize("sizes", SIZES, ids=lambda s: "+".join("%dx%d" % p for p in s))
def test_tile_order_covers_every_tile(sizes):
    r, g = _case(sizes, 8, 16, 3)
    _agree(r, g, 3)


@pytest.mark.parametrize("flags", [3, 2])
@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("F", [0, 8, 16, 32])
def test_chosen_lds_batches(F, tile, flags):
    r, g = _case([(130, 75)], F, tile, 10 + F + tile)
    _agree(r, g, flags)


@pytest.mark.parametrize("size,tile", [
    ((256, 256), 16), ((257, 256), 16),   # 256 tiles, a CU for each, and 272
    ((512, 384), 16), ((513, 384), 16),   # 768 tiles, three for each, and 792
    ((1040, 1024), 16),                   # 4160 tiles
    ((128, 128), 8), ((129, 128), 8),
], ids=str)
@pytest.mark.parametrize("F", [16, 32])
def test_lds_batches_chosen_by_tiles(F, size, tile):
    r, g = _case([size], F, tile, 20 + F)
    _agree(r, g, 3)


@pytest.mark.parametrize("batch,batch_bwd", [(64, 0), (128, 0), (256, 0), (64, 256), (128, 64), (256, 128)])
@pytest.mark.parametrize("persistent", [0, 1])
@pytest.mark.parametrize("tile,size", [(8, (40, 30)), (8, (140, 130)), (16, (40, 30)), (16, (520, 400)), (32, (40, 30))])
@pytest.mark.parametrize("F", [0, 16, 32])
def test_every_batch_a_caller_may_pass(F, tile, size, persistent, batch, batch_bwd):
    r, g = _case([size], F, tile, 30 + F + tile, lds_batch=batch, lds_batch_bwd=batch_bwd, persistent=persistent)
    _agree(r, g, 3)
