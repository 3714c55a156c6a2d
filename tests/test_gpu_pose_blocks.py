"""gs_pose_grad over its two widths of a workgroup (1024 or 512 threads for 2048
Gaussians, by Gaussians times views): the same visible Gaussians
among more and more invisible ones, at the first and last index, around the
workgroups' edges and at random.

The contributions are the same floats; they are summed in FP64 in another
order and rounded once to float32, so two splits differ by at most one
float32 rounding of the twist, 2^-23 of it, plus FP64 rounding that
cancellation can raise against a small component: 1e-6 of the twist's largest.
"""
import numpy as np
import pytest

from paper_2603_27781_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _small(n_views):
    from paper_2603_27781_amd import raster
    rng = np.random.default_rng(3)
    sc = wl.box_scene(rng, 300, (-1, -0.7, 1.5), (1, 0.7, 4), -3.2, 0.4, 0)
    views = [wl.make_view(33, 17, 26.0, wl.se3_exp(wl._random_twist(rng, 0.05, 0.05))) for _ in range(n_views)]
    g = raster.Gaussians.from_numpy(sc)
    r = raster.Rasterizer(sc.n, 0, raster.Views(views, 16), raster.Config())
    r.ensure_capacity(g)
    r.forward(g)
    go = torch.randn(r.out.shape, generator=torch.Generator("cuda").manual_seed(5), device="cuda")
    r.render_bwd(g, go, 3, g.zeros_like())
    return sc, views, g, r, r.pose_grad(g).clone()


@pytest.mark.parametrize("n,n_views", [(511, 1), (513, 1), (2047 * 512, 2), (2 << 20, 1), ((2 << 20) + 1, 1),
                                       (2_200_000, 3), (2_200_000, 64)])
def test_pose_grad_splits(n, n_views):
    from paper_2603_27781_amd import raster
    sc, views, g, r, want = _small(n_views)
    m = sc.n
    rng = np.random.default_rng(n)
    fixed = sorted({i for i in (0, n - 1, 511, 512, 1023, 1024, 2047, 2048) if i < n})
    free = rng.permutation(n)[:m]
    idx = np.unique(np.concatenate([fixed, free[~np.isin(free, fixed)]]).astype(np.int64)[:m])
    assert idx.size == m
    to = torch.from_numpy(idx).cuda()
    big = raster.Gaussians(**{k: torch.zeros(*getattr(g, k).shape[:-1], n, device="cuda")
                              for k in ("mu", "log_scale", "quat", "logit", "color", "feat")})
    for k in ("mu", "log_scale", "quat", "logit", "color", "feat"):
        getattr(big, k)[..., to] = getattr(g, k)
    R = raster.Rasterizer(n, 0, raster.Views(views, 16), raster.Config(), capacity=1024)
    touched = R.touched[: n_views * n].view(n_views, n)
    touched.zero_()
    touched[:, to] = r.touched[: n_views * m].view(n_views, m)
    geo = R.grad2d[: n_views * n * 8].view(n_views, n, 8)
    geo.fill_(float("nan"))  # unwritten where nothing is visible
    geo[:, to] = r.grad_geo
    got = R.pose_grad(big).clone()
    scale = want.abs().amax(dim=1, keepdim=True)
    assert float(scale.min()) > 0
    assert bool(((got - want).abs() <= 1e-6 * scale).all())
    if n_views < 64:  # (8 MB of partials)
        assert torch.equal(R.pose_grad(big, noalloc=True), got)


def test_workspace_grows():
    import ctypes
    from paper_2603_27781_amd import _lib
    L, b, last = _lib.load(), ctypes.c_size_t(0), {}
    for n in sorted({2 ** k + d for k in range(0, 30) for d in (-1, 0, 1) if 2 ** k + d > 0}):
        for v in (1, 2, 16, 64):
            assert L.gs_pose_grad_workspace(n, v, ctypes.byref(b)) == 0
            assert b.value >= max(last.get(v, 0), last.get(v // 2, 0) if v > 1 else 0)
            last[v] = b.value
