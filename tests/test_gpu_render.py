"""GPU parity of the forward and backward rasteriser against the FP64
oracle: pixels within 1e-4 relative (plus the cutoff ambiguity band),
gradients within 1e-3 relative."""
import math

import numpy as np
import pytest
import torch

from oracle.grads import gradients
from oracle.loss import dloss_dimg, mse
from oracle.gauss import mahalanobis_sq
from oracle.render import render_box, render_bruteforce, render_pixels
from paper_2505_09324_amd import _lib, synth
from gpu_util import (VARIANTS, GpuFrame, assert_grads_close, assert_pixels_close, dense_long_lists,
                      dev, host, loss_bound)

pytestmark = pytest.mark.gpu


def _c1():
    frame, _ = synth.make_frame(128, 128, seed=101)
    xy, chol, rgb = synth.random_gaussians(500, 128, 128, seed=102)
    return frame, xy, chol, rgb


@pytest.mark.parametrize("T,ppl", VARIANTS)
def test_forward_tiny_frame(T, ppl):
    print(f"fwd tiny T={T} ppl={ppl}", flush=True)
    frame, xy, chol, rgb = _c1()
    f = GpuFrame(128, 128, 500, T, ppl=ppl)
    img, dl, loss = f.forward(dev(xy), dev(chol), dev(rgb), dev(frame))
    ref = render_bruteforce(xy, chol, rgb, 128, 128)
    assert_pixels_close(host(img), ref)
    m = mse(ref["img"], frame)
    assert float(loss) == pytest.approx(m, rel=1e-4)
    g = dloss_dimg(ref["img"], frame)
    np.testing.assert_allclose(host(dl), g, rtol=0, atol=1e-4 * np.abs(g).max() + 1e-12)


def test_forward_single_gaussian_closed_form():
    print("fwd single", flush=True)
    l = np.array([[1.7, -0.8, 2.2]], np.float32)
    xy = np.array([[20.3, 17.9]], np.float32)
    rgb = np.array([[0.9, 0.4, -0.3]], np.float32)
    f = GpuFrame(45, 37, 1, 16)
    img, _, _ = f.forward(dev(xy), dev(l), dev(rgb))
    L = np.array([[1.7, 0.0], [-0.8, 2.2]])
    Si = np.linalg.inv(L @ L.T)
    ys, xs = np.mgrid[0:37, 0:45]
    d = np.stack([xs + 0.5 - 20.3, ys + 0.5 - 17.9], -1)
    q = np.einsum("...i,ij,...j->...", d, Si, d)
    w = np.where(q <= 9, np.exp(-q / 2), 0.0)
    for k in range(3):
        np.testing.assert_allclose(host(img)[k], rgb[0, k] * w, rtol=1e-5, atol=1e-7)


def test_forward_ragged_frame_long_lists():
    """Lists longer than one LDS chunk (dense large Gaussians) and a frame
    that is not a multiple of the tile size."""
    print("fwd long lists", flush=True)
    W, H, N = 70, 53, 1500
    xy, chol, rgb = synth.random_gaussians(N, W, H, seed=12, scale_lo=2.0, scale_hi=9.0)
    chol[:, 1] = np.random.default_rng(2).uniform(-3, 3, N).astype(np.float32)
    rgb -= 0.5
    ref = render_box(xy, chol, rgb, H, W)
    for T, ppl in VARIANTS:
        f = GpuFrame(W, H, N, T, ppl=ppl)
        b = f.bin(dev(xy), dev(chol))
        assert np.diff(b["tile_start"]).max() > 256
        img, _, _ = f.forward(dev(xy), dev(chol), dev(rgb))
        assert_pixels_close(host(img), ref, what=f"T={T} ppl={ppl}")


@pytest.mark.parametrize("T,ppl", VARIANTS)
def test_backward_tiny_frame(T, ppl):
    print(f"bwd tiny T={T} ppl={ppl}", flush=True)
    frame, xy, chol, rgb = _c1()
    chol[:, 1] = np.random.default_rng(4).uniform(-1, 1, 500).astype(np.float32)
    f = GpuFrame(128, 128, 500, T, ppl=ppl)
    dl = dloss_dimg(render_box(xy, chol, rgb, 128, 128, want_bounds=False)["img"], frame)
    f.forward(dev(xy), dev(chol), dev(rgb))
    gx, gc, gr = f.backward(dev(rgb), dev(dl.astype(np.float32)))
    ref = gradients(xy, chol, rgb, dl.astype(np.float32), 128, 128)
    assert_grads_close({"xy": host(gx), "chol": host(gc), "rgb": host(gr)}, ref)


@pytest.mark.parametrize("T,ppl", VARIANTS)
def test_forward_needles(T, ppl):
    """Thin, sheared ellipses of every sign: the sub-blocks that a row strip's
    cut of the ellipse selects hold every pixel inside the cutoff."""
    print(f"fwd needles T={T} ppl={ppl}", flush=True)
    W, H, N = 75, 67, 120
    r = np.random.default_rng(63)
    xy = (r.uniform(-0.1, 1.1, (N, 2)) * (W, H)).astype(np.float32)
    sign = r.choice([-1.0, 1.0], (N, 2))
    chol = np.stack([sign[:, 0] * r.uniform(0.3, 12, N), r.uniform(-12, 12, N),
                     sign[:, 1] * r.uniform(0.3, 2, N)], 1).astype(np.float32)
    rgb = r.uniform(-1, 1, (N, 3)).astype(np.float32)
    img, _, _ = GpuFrame(W, H, N, T, ppl=ppl).forward(dev(xy), dev(chol), dev(rgb))
    assert_pixels_close(host(img), render_box(xy, chol, rgb, H, W))


# every sub-block's list is the whole frame's: one at a time, a batch of 16
# with lanes to spare, full, and full with a rest
@pytest.mark.parametrize("T,ppl", VARIANTS)
@pytest.mark.parametrize("N", [1, 7, 8, 15, 16, 17, 24, 41])
def test_backward_list_lengths(N, T, ppl):
    print(f"bwd lists of {N} T={T} ppl={ppl}", flush=True)
    W, H = 30, 35
    xy, chol, rgb = synth.random_gaussians(N, W, H, seed=60 + N, scale_lo=20.0, scale_hi=30.0)
    chol[:, 1] = np.random.default_rng(N).uniform(-5, 5, N).astype(np.float32)
    rgb -= 0.5
    dl = np.random.default_rng(61).standard_normal((3, H, W)).astype(np.float32)
    f = GpuFrame(W, H, N, T, ppl=ppl)
    f.bin(dev(xy), dev(chol))
    gx, gc, gr = f.backward(dev(rgb), dev(dl))
    ref = gradients(xy, chol, rgb, dl, H, W)
    assert_grads_close({"xy": host(gx), "chol": host(gc), "rgb": host(gr)}, ref)


def test_backward_long_lists():
    print("bwd long lists", flush=True)
    W, H, N = 64, 48, 1200
    xy, chol, rgb = synth.random_gaussians(N, W, H, seed=13, scale_lo=2.0, scale_hi=8.0)
    chol[:, 1] = np.random.default_rng(7).uniform(-2, 2, N).astype(np.float32)
    target = np.random.default_rng(8).uniform(0, 1, (3, H, W)).astype(np.float32)
    dl = dloss_dimg(render_box(xy, chol, rgb, H, W, want_bounds=False)["img"], target).astype(np.float32)
    ref = gradients(xy, chol, rgb, dl, H, W)
    for T, ppl in VARIANTS:
        f = GpuFrame(W, H, N, T, ppl=ppl)
        f.forward(dev(xy), dev(chol), dev(rgb))
        gx, gc, gr = f.backward(dev(rgb), dev(dl))
        assert_grads_close({"xy": host(gx), "chol": host(gc), "rgb": host(gr)}, ref)


def test_full_hd_sampled_pixels_and_gaussians():
    """1920x1080, 30k Gaussians, in the tile configuration the fitter uses:
    2000 sampled pixels against the per-pixel oracle; gradients of 24 sampled
    Gaussians against the oracle evaluated on their windows."""
    print("1080p sampled", flush=True)
    W, H, N = 1920, 1080, 30000
    frame, _ = synth.make_frame(W, H, seed=201)
    xy, chol, rgb = synth.random_gaussians(N, W, H, seed=202, scale_lo=1.0, scale_hi=8.0)
    chol[:, 1] = np.random.default_rng(9).uniform(-2, 2, N).astype(np.float32)
    f = GpuFrame(W, H, N, 16)
    img, dl, _ = f.forward(dev(xy), dev(chol), dev(rgb), dev(frame))
    rng = np.random.default_rng(10)
    px = rng.integers(0, W, 2000)
    py = rng.integers(0, H, 2000)
    ref = render_pixels(xy, chol, rgb, px, py)
    assert_pixels_close(host(img)[:, py, px], ref)
    # gradients of sampled Gaussians: oracle image on each window, then the
    # oracle gradient of that Gaussian with dL/dC from the oracle image
    gx, gc, gr = f.backward(dev(rgb), dl)
    _check_window_grads(xy, chol, rgb, frame, (gx, gc, gr), rng.choice(N, 24, replace=False))


def _check_window_grads(xy, chol, rgb, frame, grads, sel):
    """Gradients of Gaussians `sel` against the oracle: the oracle image on a
    window round each one's 3-sigma box, dL/dC of the whole-frame MSE there,
    and the oracle gradient of that one Gaussian."""
    H, W = frame.shape[1:]
    gx, gc, gr = (host(g) for g in grads)
    for n in sel:
        l1, l2, l3 = chol[n].astype(np.float64)
        rx, ry = 3 * abs(l1), 3 * math.hypot(l2, l3)
        x0, x1 = max(0, int(xy[n, 0] - rx) - 2), min(W, int(xy[n, 0] + rx) + 3)
        y0, y1 = max(0, int(xy[n, 1] - ry) - 2), min(H, int(xy[n, 1] + ry) + 3)
        if x1 <= x0 or y1 <= y0:
            continue
        ys, xs = np.mgrid[y0:y1, x0:x1]
        win = render_pixels(xy, chol, rgb, xs.ravel(), ys.ravel())["img"].reshape(3, y1 - y0, x1 - x0)
        full_dl = 2.0 * (win - frame[:, y0:y1, x0:x1]) / (3.0 * W * H)
        sub_xy = xy[n:n + 1] - np.array([x0, y0], np.float32)
        r = gradients(sub_xy, chol[n:n + 1], rgb[n:n + 1], full_dl, y1 - y0, x1 - x0)
        assert_grads_close({"xy": gx[n:n + 1], "chol": gc[n:n + 1], "rgb": gr[n:n + 1]}, r)


def test_maximum_sizes_forward_backward_fused():
    """The largest shape the 16-bit tile and id key fields hold: N = 65536
    Gaussians on 2048x2048 at T = 8 (256 x 256 = 65536 tiles), with the last
    Gaussian in the last tile.  Sampled pixels (and the last tile's) against
    the per-pixel oracle; render_bwd and the fused pass against the oracle's
    gradients of sampled Gaussians, the last one included; the fused loss
    against the oracle's MSE."""
    print("maximum sizes render", flush=True)
    W = H = 2048
    N = 65536
    frame, _ = synth.make_frame(W, H, seed=303)
    xy, chol, rgb = synth.random_gaussians(N, W, H, seed=301, scale_lo=0.3, scale_hi=2.0)
    xy[-1] = [W - 2.75, H - 1.5]
    f = GpuFrame(W, H, N, 8)
    P = [dev(xy), dev(chol), dev(rgb)]
    img, dl, loss = f.forward(*P, dev(frame))
    rng = np.random.default_rng(304)
    ys, xs = np.mgrid[H - 8:H, W - 8:W]
    px = np.concatenate([rng.integers(0, W, 300), xs.ravel()])
    py = np.concatenate([rng.integers(0, H, 300), ys.ravel()])
    assert_pixels_close(host(img)[:, py, px], render_pixels(xy, chol, rgb, px, py))
    full = render_box(xy, chol, rgb, W, H, want_bounds=False)["img"]
    assert float(loss) == pytest.approx(mse(full, frame), rel=1e-4)
    sel = np.concatenate([rng.choice(N - 1, 12, replace=False), [N - 1]])
    _check_window_grads(xy, chol, rgb, frame, f.backward(P[2], dl), sel)
    g = [torch.zeros(N, d, device="cuda") for d in (2, 3, 3)]
    floss = torch.empty((), device="cuda")
    _lib.render_fused(f.shape, f.ws, P[2], dev(frame), *g, loss=floss)
    torch.cuda.synchronize()
    assert float(floss) == pytest.approx(mse(full, frame), rel=1e-4)
    _check_window_grads(xy, chol, rgb, frame, g, sel)


def _marginal_gaussians(W, H, sbh, n, seed):
    """n sheared Gaussians of mixed orientation, each with its mean outside
    one 8 x sbh pixel block and its cutoff ellipse reaching that block only
    just: the smallest q over the block's in-frame pixel centres lies 5e-4
    to 4e-3 below 9 (FP64, on the FP32 parameters)."""
    rng = np.random.default_rng(seed)
    xy = np.zeros((n, 2), np.float32)
    chol = np.zeros((n, 3), np.float32)
    k = 0
    while k < n:
        bx, by = int(rng.integers(0, -(-W // 8))), int(rng.integers(0, -(-H // sbh)))
        xs = np.arange(bx * 8, min(W, bx * 8 + 8)) + 0.5
        ys = np.arange(by * sbh, min(H, by * sbh + sbh)) + 0.5
        l = np.array([rng.uniform(0.4, 3.0) * rng.choice([-1.0, 1.0]), rng.uniform(-4.0, 4.0),
                      rng.uniform(0.4, 3.0)])
        side = [xs[0] - rng.uniform(0.2, 6.0), xs[-1] + rng.uniform(0.2, 6.0),
                rng.uniform(xs[0], xs[-1])]
        cx = side[rng.integers(0, 3)]
        side = [ys[0] - rng.uniform(0.2, 6.0), ys[-1] + rng.uniform(0.2, 6.0),
                rng.uniform(ys[0], ys[-1])]
        cy = side[rng.integers(0, 3)]
        if xs[0] <= cx <= xs[-1] and ys[0] <= cy <= ys[-1]:
            continue
        X, Y = np.meshgrid(xs, ys)
        qmin = mahalanobis_sq(X - cx, Y - cy, *l).min()
        l *= math.sqrt(qmin / rng.uniform(9.0 - 3e-3, 9.0 - 1e-3))  # q scales as 1 / s^2
        mu, lf = np.array([cx, cy], np.float32), l.astype(np.float32)
        q32 = mahalanobis_sq(X - float(mu[0]), Y - float(mu[1]), *lf.astype(np.float64)).min()
        if not 9.0 - 4e-3 <= q32 <= 9.0 - 5e-4:
            continue
        xy[k], chol[k] = mu, lf
        k += 1
    return xy, chol


@pytest.mark.parametrize("T,ppl", VARIANTS)
def test_block_masks_keep_marginal_pixels(T, ppl):
    """Gaussians whose cutoff ellipse reaches a neighbouring 8 x 8P pixel
    block only just, on a ragged 123 x 90 frame: pixels and fused-pass
    gradients against the oracle.  A block dropped by the staging's
    ellipse test would lose an exp(-4.5) c' contribution, far above the
    pixel tolerance (the marginal q lie outside the oracle's ambiguity
    band)."""
    print(f"marginal blocks T={T} ppl={ppl}", flush=True)
    W, H, N = 123, 90, 300
    xy, chol = _marginal_gaussians(W, H, 8 * ppl, N, seed=400 + 10 * T + ppl)
    rgb = np.random.default_rng(401).uniform(0.2, 1.0, (N, 3)).astype(np.float32)
    frame, _ = synth.make_frame(W, H, seed=402)
    f = GpuFrame(W, H, N, T, ppl=ppl)
    P = [dev(xy), dev(chol), dev(rgb)]
    img, _, _ = f.forward(*P, dev(frame))
    ref = render_bruteforce(xy, chol, rgb, H, W)
    assert_pixels_close(host(img), ref)
    g = [torch.zeros(N, d, device="cuda") for d in (2, 3, 3)]
    _lib.render_fused(f.shape, f.ws, P[2], dev(frame), *g)
    torch.cuda.synchronize()
    want = gradients(xy, chol, rgb, dloss_dimg(ref["img"], frame), H, W)
    assert_grads_close({"xy": host(g[0]), "chol": host(g[1]), "rgb": host(g[2])}, want)


@pytest.mark.parametrize("T,ppl", VARIANTS)
def test_fused_render_matches_oracle_and_counts_pairs(T, ppl):
    """Fused forward+MSE+backward: loss and accumulated gradients vs the
    oracle; the in-cutoff pair count vs the oracle's count."""
    print(f"fused T={T} ppl={ppl}", flush=True)
    from oracle.render import count_pairs_in_cutoff
    frame, xy, chol, rgb = _c1()
    chol[:, 1] = np.random.default_rng(4).uniform(-1, 1, 500).astype(np.float32)
    f = GpuFrame(128, 128, 500, T, ppl=ppl)
    P = [dev(xy), dev(chol), dev(rgb)]
    _lib.project_bin(f.shape, P[0], P[1], f.ws)
    g = [torch.zeros(500, d, device="cuda") for d in (2, 3, 3)]
    loss = torch.empty((), device="cuda")
    _lib.render_fused(f.shape, f.ws, P[2], dev(frame), *g, loss=loss)
    torch.cuda.synchronize()
    img = render_box(xy, chol, rgb, 128, 128, want_bounds=False)["img"]
    assert float(loss) == pytest.approx(mse(img, frame), rel=1e-4)
    ref = gradients(xy, chol, rgb, dloss_dimg(img, frame), 128, 128)
    assert_grads_close({"xy": host(g[0]), "chol": host(g[1]), "rgb": host(g[2])}, ref)
    # accumulation: a second call doubles the gradients
    _lib.render_fused(f.shape, f.ws, P[2], dev(frame), *g)
    torch.cuda.synchronize()
    assert_grads_close({"xy": host(g[0]) / 2, "chol": host(g[1]) / 2, "rgb": host(g[2]) / 2}, ref)
    # pairs whose q lies within 1e-4 of the cutoff may fall either way
    got, want = _lib.count_pairs(f.shape, f.ws), count_pairs_in_cutoff(xy, chol, 128, 128)
    assert abs(got - want) <= 2, (got, want)


def test_fused_long_lists_every_variant():
    """The fused pass on lists longer than 256 and 512 (the staged-twice
    branch: forward over every chunk, residuals, then each chunk staged again
    for the backward and flushed): loss and every gradient element against
    the oracle, for every (tile, pixels per lane) variant."""
    W, H, N, frame, xy, chol, rgb = dense_long_lists()
    ref = render_box(xy, chol, rgb, H, W)
    want_loss = mse(ref["img"], frame)
    tol = loss_bound(ref, frame)
    want = gradients(xy, chol, rgb, dloss_dimg(ref["img"], frame), H, W)
    P = [dev(xy), dev(chol), dev(rgb)]
    for T, ppl in VARIANTS:
        print(f"fused long lists T={T} ppl={ppl}", flush=True)
        f = GpuFrame(W, H, N, T, ppl=ppl)
        b = f.bin(P[0], P[1])
        lens = np.diff(b["tile_start"])
        assert lens.max() > 512 and (lens > 256).sum() >= 9
        g = [torch.zeros(N, d, device="cuda") for d in (2, 3, 3)]
        loss = torch.empty((), device="cuda")
        _lib.render_fused(f.shape, f.ws, P[2], dev(frame), *g, loss=loss)
        torch.cuda.synchronize()
        assert abs(float(loss) - want_loss) <= tol, (float(loss), want_loss, tol)
        assert_grads_close({"xy": host(g[0]), "chol": host(g[1]), "rgb": host(g[2])}, want)


@pytest.mark.parametrize("W,H", [(400, 300), (600, 400), (640, 400), (1100, 1000)])
def test_every_route_at_frame_sizes(W, H):
    """Frames whose number of sub-blocks makes four, two or one wavefront
    share a sub-block (every variant meets all three over the sizes), with
    800 of 1500 Gaussians in one corner so that its lists take several LDS
    chunks: pixels, losses and the gradients of both backward passes against
    the oracle."""
    N = 1500
    xy, chol, rgb = synth.random_gaussians(N, W, H, seed=61, scale_lo=1.0, scale_hi=8.0)
    xy[:800] = 20.0 + xy[:800] * (40.0 / W)
    chol[:, 1] = np.random.default_rng(62).uniform(-3, 3, N).astype(np.float32)
    rgb -= 0.5
    frame, _ = synth.make_frame(W, H, seed=63)
    ref = render_box(xy, chol, rgb, H, W)
    want_loss, tol = mse(ref["img"], frame), loss_bound(ref, frame)
    dl = dloss_dimg(ref["img"], frame)
    want = gradients(xy, chol, rgb, dl, H, W)
    P = [dev(xy), dev(chol), dev(rgb)]
    for T, ppl in VARIANTS:
        print(f"routes {W}x{H} T={T} ppl={ppl}", flush=True)
        f = GpuFrame(W, H, N, T, max_pairs=400000, ppl=ppl)
        img, _, loss = f.forward(*P, dev(frame))
        assert_pixels_close(host(img), ref, what=f"T={T} ppl={ppl}")
        g = [torch.zeros(N, d, device="cuda") for d in (2, 3, 3)]
        floss = torch.empty((), device="cuda")
        _lib.render_fused(f.shape, f.ws, P[2], dev(frame), *g, loss=floss)
        b = f.backward(P[2], dev(dl.astype(np.float32)))
        for x in (loss, floss):
            assert abs(float(x) - want_loss) <= tol, (float(x), want_loss, tol)
        for grads in (g, b):
            assert_grads_close(dict(zip(("xy", "chol", "rgb"), map(host, grads))), want)


@pytest.mark.parametrize("tile", [8, 16, 32])
def test_counted_pairs_are_the_rendered_ones(tile):
    """One Gaussian per 16x16 block with its cutoff through the centre of a
    pixel (q = 9 there to a few roundings), colour 1: the pixels with a value
    are the pairs that count_pairs finds, to the last borderline one."""
    print(f"counted pairs tile={tile}", flush=True)
    W, H = 1280, 720
    rng = np.random.default_rng(11)
    c = np.arange((W // 16) * (H // 16))
    xy = np.stack([c % (W // 16) * 16 + 8 + rng.uniform(-1, 1, len(c)),
                   c // (W // 16) * 16 + 8 + rng.uniform(-1, 1, len(c))], 1).astype(np.float32)
    px = np.floor(xy) + 0.5 + rng.integers(-3, 4, xy.shape)
    d = px - xy.astype(np.float64)
    l2 = rng.uniform(-0.3, 0.3, len(c))
    l1 = rng.uniform(1.0, 1.3, len(c))
    # l3 for q = 9 at (dx, dy); where that is no Gaussian of the block, a round one
    l3 = np.abs(d[:, 1] - l2 * d[:, 0] / l1) / np.sqrt(np.maximum(9 - (d[:, 0] / l1) ** 2, 1e-3))
    round_ = (l3 < 0.3) | (l3 > 1.4)
    l2[round_], l1[round_] = 0.0, np.hypot(d[round_, 0], d[round_, 1]) / 3
    l3[round_] = l1[round_]
    chol = np.stack([l1, l2, l3], 1).astype(np.float32)
    N = len(c)
    f = GpuFrame(W, H, N, tile)
    img, _, _ = f.forward(dev(xy), dev(chol), torch.ones(N, 3, device="cuda"))
    pairs = _lib.count_pairs(f.shape, f.ws)
    assert pairs > 20 * N
    assert int((img[0] != 0).sum()) == pairs


# size -> variants rendered at it; together every (variant, share) pair of the
# raster: four, two or one wavefront on a sub-block
ROUTES = {
    (320, 240): VARIANTS,
    (480, 400): [(8, 1), (16, 1), (32, 1)],
    (640, 480): VARIANTS[:5],
    (960, 720): [(16, 2), (32, 2), (32, 4)],
    (1100, 1000): [(32, 4)],
}


@pytest.mark.parametrize("W,H", ROUTES)
def test_every_variant_with_every_share(W, H):
    """As the frames above, at the sizes of ROUTES; the rule that picks the
    share is read from the source, and the pairs visited must be complete."""
    import pathlib
    import re
    src = pathlib.Path(_lib.HERE, "csrc", "raster_tile.h").read_text()
    four, two = map(int, re.search(r"sub_blocks <= (\d+) \? 4 : sub_blocks <= (\d+) \? 2 : 1",
                                   src).groups())

    def share(w, h, T, ppl):
        n = -(-w // T) * -(-h // T) * (T // 8) * (T // (8 * ppl))
        return 4 if n <= four else 2 if n <= two else 1

    visited = {(v, share(w, h, *v)) for (w, h), vs in ROUTES.items() for v in vs}
    assert visited == {(v, s) for v in VARIANTS for s in (4, 2, 1)}
    N = 1500
    xy, chol, rgb = synth.random_gaussians(N, W, H, seed=61, scale_lo=1.0, scale_hi=8.0)
    xy[:800] = 20.0 + xy[:800] * (40.0 / W)
    chol[:, 1] = np.random.default_rng(62).uniform(-3, 3, N).astype(np.float32)
    rgb -= 0.5
    frame, _ = synth.make_frame(W, H, seed=63)
    ref = render_box(xy, chol, rgb, H, W)
    want_loss, tol = mse(ref["img"], frame), loss_bound(ref, frame)
    dl = dloss_dimg(ref["img"], frame)
    want = gradients(xy, chol, rgb, dl, H, W)
    P = [dev(xy), dev(chol), dev(rgb)]
    for T, ppl in ROUTES[W, H]:
        print(f"shares {W}x{H} T={T} ppl={ppl} share={share(W, H, T, ppl)}", flush=True)
        f = GpuFrame(W, H, N, T, max_pairs=400000, ppl=ppl)
        img, _, loss = f.forward(*P, dev(frame))
        assert_pixels_close(host(img), ref, what=f"T={T} ppl={ppl}")
        g = [torch.zeros(N, d, device="cuda") for d in (2, 3, 3)]
        floss = torch.empty((), device="cuda")
        _lib.render_fused(f.shape, f.ws, P[2], dev(frame), *g, loss=floss)
        b = f.backward(P[2], dev(dl.astype(np.float32)))
        for x in (loss, floss):
            assert abs(float(x) - want_loss) <= tol, (float(x), want_loss, tol)
        for grads in (g, b):
            assert_grads_close(dict(zip(("xy", "chol", "rgb"), map(host, grads))), want)
