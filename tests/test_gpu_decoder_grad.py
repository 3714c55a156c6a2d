"""Decoder gradients of the SLAM loss at the class counts where the kernel's
loops and tiles end (groups of four classes, 16-class operand tiles, the
three tile counts), for each feature count, with and without the mask, and
pixel counts that leave a last workgroup nearly empty or put two views in
one, against FP64 autograd on the CPU.

Tolerance: the per-pixel softmax is binary32 (hardware exp, about 1e-6
relative; BCE's 1 - p loses up to 1 / (1 - p) of it, p < 0.99 here), the sums
of at least 64 pixels are FP64: 2e-5 of the tensor's maximum for the
cross-entropy, 2e-4 for the BCE."""
import ctypes

import numpy as np
import pytest

from paper_2603_27781_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _want(F, f, labels, W, b, M, sizes, w_sem, bce):
    W = W.double().requires_grad_(True)
    b = b.double().requires_grad_(True)
    f = f.double().requires_grad_(True)
    z = f.T @ W + b
    lp = torch.log_softmax(z, 1)
    y = labels.long()[:, None]
    if bce:
        q = torch.log1p(-torch.softmax(z, 1)).clamp(min=-100.0)
        S = -q.scatter(1, y, lp.gather(1, y).clamp(min=-100.0)).sum(1)
    else:
        S = -lp.gather(1, y)[:, 0]
    inv = torch.cat([torch.full((w * h,), 1.0 / (w * h), dtype=torch.float64) for w, h in sizes])
    term = w_sem * (S * M.double() * inv).sum()
    term.backward()
    if W.shape[1] == 1:  # p = 1: nothing to learn (autograd of the clamped log(1 - p) at 0 has no value)
        return 0.0, torch.zeros_like(f), torch.zeros_like(W), torch.zeros_like(b)
    return float(term.detach()), f.grad, W.grad, b.grad


@pytest.mark.parametrize("bce", [False, True])
@pytest.mark.parametrize("F,K", [(8, 1), (8, 3), (8, 4), (8, 5), (8, 17), (16, 2), (16, 15), (16, 16), (16, 17), (16, 20),
                                 (16, 31), (16, 32), (16, 33), (16, 64), (32, 1), (32, 16), (32, 18), (32, 33), (32, 63),
                                 (32, 64)])
def test_decoder_gradients(F, K, bce):
    from paper_2603_27781_amd import _lib, raster
    g = torch.Generator().manual_seed(1000 * F + K)
    sizes = [(33, 31), (7, 5), (40, 30)] if K % 2 else [(257, 1)]
    P = sum(w * h for w, h in sizes)
    masked = K % 3 == 0
    views = [wl.make_view(w, h, 50.0, np.eye(4)) for w, h in sizes]
    r = raster.Rasterizer(1, F, raster.Views(views, 16), raster.Config(), capacity=64)
    out = torch.rand(5 + F, P, generator=g)
    out[4] = 1.0
    out[5:] = torch.randn(F, P, generator=g)
    dep = out[3] + 0.1 * torch.rand(P, generator=g)
    labels = torch.randint(0, K, (P,), generator=g, dtype=torch.int32)
    W, b = torch.randn(F, K, generator=g) / F ** 0.5, 0.1 * torch.randn(K, generator=g)
    r.out.copy_(out)
    o = _lib.GsSlamLossOpts()
    _lib.check(_lib.load().gs_default_slam_loss_opts(ctypes.byref(o)), "opts")
    o.ssim_lambda, o.obs_factor = 0.0, 1.0  # with the mask: only residuals below the median count
    o.flags = (_lib.GS_LOSS_OBS_MASK if masked else 0) | (_lib.GS_LOSS_BCE if bce else 0)
    Wd, bd = W.cuda(), b.cuda()
    r.slam_loss(torch.rand(3, P, generator=g).cuda(), dep.cuda(), labels.cuda(), Wd, o, bias=bd, decoder_grads=True)
    torch.cuda.synchronize()
    M = (r.masks.cpu() & 1) if masked else torch.ones(P)
    assert not masked or 0 < int(M.sum()) < P
    term, gf, gW, gb = _want(F, out[5:], labels, W, b, M, sizes, float(np.float32(o.w_sem)), bce)
    tol = 2e-4 if bce else 2e-5
    assert abs(float(r.slam_terms[3]) - term) <= tol * max(abs(term), 1e-9)
    for got, want in ((r.grad_out[5:], gf), (r.grad_decoder_w, gW), (r.grad_decoder_b, gb)):
        got, top = got.cpu().double(), float(want.abs().max())
        # one class: every gradient is exactly 0 up to rounding of the softmax
        assert float((got - want).abs().max()) <= tol * max(top, 1e-9), (float((got - want).abs().max()), top)


@pytest.mark.parametrize("bce", [False, True])
@pytest.mark.parametrize("K", [5, 6, 7, 8, 50])
def test_labels_outside_the_classes_are_no_class(K, bce):
    """Labels -1 and K .. K + 3 (void pixels) are no class: a BCE term has the
    other classes' logarithms only, a cross-entropy none, and the gradients
    are those of a softmax no class of which is the label; the features' equal
    those of the call without decoder gradients.  1e-5 relative between the two
    variants (the same binary32 formulas, summed differently), against FP64 the
    tolerances above."""
    from paper_2603_27781_amd import _lib, raster
    F, P = 16, 300
    g = torch.Generator().manual_seed(K)
    r = raster.Rasterizer(1, F, raster.Views([wl.make_view(P, 1, 50.0, np.eye(4))], 16), raster.Config(), capacity=64)
    r.out.copy_(torch.randn(5 + F, P, generator=g))
    rgb, dep = torch.rand(3, P, generator=g).cuda(), torch.rand(P, generator=g).cuda()
    labels = torch.arange(P, dtype=torch.int32) % (K + 5) - 1
    W, b = torch.randn(F, K, generator=g) / 4, 0.1 * torch.randn(K, generator=g)
    o = _lib.GsSlamLossOpts()
    _lib.check(_lib.load().gs_default_slam_loss_opts(ctypes.byref(o)), "opts")
    o.ssim_lambda, o.flags = 0.0, _lib.GS_LOSS_BCE if bce else 0
    grads, terms = [], []
    for dec in (False, True):
        r.slam_loss(rgb, dep, labels.cuda(), W.cuda(), o, bias=b.cuda(), decoder_grads=dec)
        torch.cuda.synchronize()
        grads.append(r.grad_out.cpu().clone())
        terms.append(float(r.slam_terms[3]))
    assert float((grads[0] - grads[1]).abs().max()) <= 1e-5 * float(grads[0].abs().max())
    z = r.out[5:].cpu().double().T @ W.double() + b.double()
    p = torch.softmax(z, 1)
    y = torch.zeros(P, K).double()
    has = (labels >= 0) & (labels < K)
    y[has] = torch.nn.functional.one_hot(labels[has].long(), K).double()
    S = -(y * p.log() + ((1 - y) * (1 - p).log() if bce else 0)).sum()
    dp = -y / p + (1 - y) / (1 - p)
    dz = p * (dp - (p * dp).sum(1, keepdim=True)) if bce else p - y
    w, tol = float(np.float32(o.w_sem)) / P, 2e-4 if bce else 2e-5
    assert terms[1] == pytest.approx(w * float(S), rel=tol)
    if bce:
        assert terms[0] == pytest.approx(terms[1], rel=1e-5)
    gW = w * r.out[5:].cpu().double() @ dz
    assert float((r.grad_decoder_w.cpu().double() - gW).abs().max()) <= tol * float(gW.abs().max())


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("K", [5, 6, 7, 8])
def test_features_that_are_not_finite(K, value):
    """The BCE term of a pixel with such a feature counts its K classes only,
    as without decoder gradients (1e-5 relative: the same binary32 formulas
    per pixel, summed in FP64)."""
    from paper_2603_27781_amd import _lib, raster
    F, P = 8, 300
    g = torch.Generator().manual_seed(K)
    r = raster.Rasterizer(1, F, raster.Views([wl.make_view(P, 1, 50.0, np.eye(4))], 16), raster.Config(), capacity=64)
    r.out.copy_(torch.randn(5 + F, P, generator=g))
    r.out[6, 100] = value
    rgb, dep = torch.rand(3, P, generator=g).cuda(), torch.rand(P, generator=g).cuda()
    labels = torch.randint(0, K, (P,), generator=g, dtype=torch.int32).cuda()
    W = (torch.randn(F, K, generator=g) / 4).cuda()
    o = _lib.GsSlamLossOpts()
    _lib.check(_lib.load().gs_default_slam_loss_opts(ctypes.byref(o)), "opts")
    o.ssim_lambda, o.flags = 0.0, _lib.GS_LOSS_BCE
    terms, grads = [], []
    for dec in (False, True):
        r.slam_loss(rgb, dep, labels, W, o, decoder_grads=dec)
        torch.cuda.synchronize()
        terms.append(r.slam_terms.cpu().clone())
        grads.append(r.grad_out.cpu().clone())
    assert torch.isfinite(terms[0]).all()
    assert float((terms[0] - terms[1]).abs().max()) <= 1e-5 * float(terms[0].abs().max())
    assert torch.equal(torch.isfinite(grads[0]), torch.isfinite(grads[1]))
