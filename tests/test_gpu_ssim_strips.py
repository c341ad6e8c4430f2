"""Structural-similarity kernel at the edges of its strips and row groups.

A workgroup writes a strip of 44, 108 or 236 columns at most and a multiple of
four rows of a plane; shapes on both sides of those lines, of several
workgroups per column and of widths that are no multiple of four (scalar
writes instead of groups of four) are compared with the FP64 oracle, at the
bounds of the other shapes: the sums of 121 products of FP32 numbers below one
are good to 121 * 2^-24 = 7e-6, and to 1e-5 where the terms of both signs of a
view's mean average out; a gradient takes two of them, divided by C2 = 9e-4 or
more, to 1e-3 of the larger gradients."""
import numpy as np
import pytest
import torch

from oracle import ssim as OS
from paper_2504_02437_amd import raster as R
from test_gpu_ssim import _check, _colour, _gpu, _pair

pytestmark = pytest.mark.gpu


def _views(H, W):
    """Views enough for the strips: small inputs are taken in tiles."""
    tiles = 3 * ((W + 63) // 64) * ((H + 15) // 16)
    return (601 if W <= 256 else 257) // tiles + 1


SHAPES = [(_views(H, W), 3, H, W) for H, W in (
    (11, 44), (12, 45), (13, 88), (5, 108), (16, 109), (31, 216), (33, 217),
    (9, 236), (50, 237), (150, 473), (330, 44))]
# Both sides of the lines between tiles and strips.
SHAPES += [(1, 3, 250, 344), (1, 3, 257, 344), (5, 3, 160, 256),
           (5, 3, 161, 256)]


@pytest.mark.parametrize("shape", SHAPES)
def test_strip_edges_against_the_oracle(shape):
    x, y = _pair(11, shape)
    print("case ssim strip", shape, flush=True)
    _check(x, y)


@pytest.mark.parametrize("shape", SHAPES)
def test_strip_edges_fused_equals_l1_then_ssim(shape):
    x, y = _pair(12, shape)
    print("case colour strip", shape, flush=True)
    a = _colour(x, y, 0.8, 0.2, False)
    b = _colour(x, y, 0.8, 0.2, True)
    assert b[0] == pytest.approx(a[0], rel=1e-6)
    np.testing.assert_allclose(b[1], a[1], rtol=1e-12)
    np.testing.assert_allclose(b[2], a[2], rtol=1e-12)
    np.testing.assert_array_equal(b[3], a[3])


@pytest.mark.parametrize("which", range(3))
def test_misaligned_images(which):
    """One of the three images four bytes off a 16-byte line: the same
    gradient as aligned (the same sums, written one by one)."""
    shape = (_views(21, 240), 3, 21, 240)
    x, y = _pair(13, shape)
    n = x.size
    buf = [torch.zeros(n + 4, device="cuda") for _ in range(3)]
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    ref = _colour(x, y, 0.8, 0.2, True)
    t = [b[int(i == which):][:n].view(shape) for i, b in enumerate(buf)]
    t[0].copy_(torch.from_numpy(x))
    t[1].copy_(torch.from_numpy(y))
    print("case colour misaligned", which, flush=True)
    R.loss_colour(t[0], t[1], 0.8, 0.2, t[2], loss)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(t[2].cpu().numpy(), ref[3])
    assert all(float(b[-1]) == 0.0 for b in buf)


@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("at", [(37, 120), (0, 0), (43, 1)])
def test_a_value_that_is_not_finite_stays_in_its_windows(at, value):
    """A gradient depends on the pixels at most ten rows and columns away:
    NaN there, and bit for bit as without the value further off."""
    x, y = _pair(14, (_views(61, 250), 3, 61, 250))
    good = _colour(x, y, 0.8, 0.2, True)[3][0, 1]
    x[0, 1, at[0], at[1]] = value
    print("case colour not finite", at, value, flush=True)
    loss, _, _, g = _colour(x, y, 0.8, 0.2, True)
    r, c = np.mgrid[0:61, 0:250]
    near = np.maximum(abs(r - at[0]), abs(c - at[1])) <= 10
    assert np.isnan(loss)
    assert np.isnan(g[0, 1][near]).all()
    np.testing.assert_array_equal(g[0, 1][~near], good[~near])
    assert np.isfinite(g[0, 0]).all() and np.isfinite(g[0, 2]).all()
    assert np.isfinite(g[1:]).all()


@pytest.mark.parametrize("shape", [(_views(30, 300), 3, 30, 300), (1, 3, 9, 45)])
@pytest.mark.parametrize("fused", [False, True])
def test_gradient_written_over_the_rendering(shape, fused):
    """dL in the memory of the rendered images: as with memory of its own."""
    x, y = _pair(15, shape)
    xd, yd = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    own = xd.clone()
    loss = torch.zeros(2, dtype=torch.float64, device="cuda")
    print("case colour in place", shape, fused, flush=True)
    if fused:
        R.loss_colour(xd, yd, 0.8, 0.2, own, loss[:1])
        R.loss_colour(xd, yd, 0.8, 0.2, xd, loss[1:])
    else:
        R.loss_ssim(xd, yd, 0.2, own, loss[:1])
        R.loss_ssim(xd, yd, 0.2, xd, loss[1:])
    torch.cuda.synchronize()
    np.testing.assert_array_equal(xd.cpu().numpy(), own.cpu().numpy())
    assert float(loss[0]) == pytest.approx(float(loss[1]), rel=1e-9)


# Always taken in strips: past 256 tiles, more than 64 of them in a plane; or
# more than 3,000 in all.
STRIPS = (1, 3, 250, 344)
MANY = [(3000 // (3 * ((W + 63) // 64) * ((H + 15) // 16)) + 1, 3, H, W)
        for H, W in ((11, 44), (12, 45), (13, 88), (16, 109), (33, 217),
                     (50, 237), (330, 44))]


@pytest.mark.parametrize("shape", MANY)
def test_strip_edges_of_many_views(shape):
    """Views enough for strips whatever the width fills: the first, one in the
    middle and the last against the oracle."""
    x, y = _pair(19, shape)
    print("case ssim many", shape, flush=True)
    loss, ssim, g = _gpu(x, y, 0.2)
    ref_ssim = OS.ssim_map(x, y).reshape(shape[0], -1).mean(1)
    assert np.abs(ssim - ref_ssim).max() <= 1e-5
    assert loss == pytest.approx(0.2 * np.sum(1.0 - ref_ssim), rel=1e-5)
    for k in (0, shape[0] // 2, shape[0] - 1):
        ref = OS.loss_ssim(x[k:k + 1].astype(np.float64), y[k:k + 1], 0.2)[1]
        tol = 1e-3 * np.maximum(np.abs(ref), 1e-2 * np.abs(ref).max()) + 1e-30
        assert np.all(np.abs(g[k:k + 1] - ref) <= tol)


@pytest.mark.parametrize("which", range(3))
def test_misaligned_strips(which):
    """test_misaligned_images at a size that is always taken in strips."""
    x, y = _pair(20, STRIPS)
    n = x.size
    buf = [torch.zeros(n + 4, device="cuda") for _ in range(3)]
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    ref = _colour(x, y, 0.8, 0.2, True)
    t = [b[int(i == which):][:n].view(STRIPS) for i, b in enumerate(buf)]
    t[0].copy_(torch.from_numpy(x))
    t[1].copy_(torch.from_numpy(y))
    print("case colour misaligned strips", which, flush=True)
    R.loss_colour(t[0], t[1], 0.8, 0.2, t[2], loss)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(t[2].cpu().numpy(), ref[3])
    assert all(float(b[-1]) == 0.0 for b in buf)


@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("at", [(37, 120), (0, 0), (249, 1), (120, 343)])
def test_a_value_that_is_not_finite_stays_in_its_windows_of_strips(at, value):
    x, y = _pair(21, STRIPS)
    good = _colour(x, y, 0.8, 0.2, True)[3][0, 1]
    x[0, 1, at[0], at[1]] = value
    print("case strips not finite", at, value, flush=True)
    loss, _, _, g = _colour(x, y, 0.8, 0.2, True)
    r, c = np.mgrid[0:STRIPS[2], 0:STRIPS[3]]
    near = np.maximum(abs(r - at[0]), abs(c - at[1])) <= 10
    assert np.isnan(loss)
    assert np.isnan(g[0, 1][near]).all()
    np.testing.assert_array_equal(g[0, 1][~near], good[~near])
    assert np.isfinite(g[0, 0]).all() and np.isfinite(g[0, 2]).all()


@pytest.mark.parametrize("shape", [STRIPS, (1, 3, 61, 90)])
@pytest.mark.parametrize("value", [1e19, -1e20, 1.5e20])
def test_a_value_whose_square_runs_over(shape, value):
    """Finite in both forms (strips, tiles): the windows that hold it have an
    SSIM of 0 and pass no gradient."""
    x, y = _pair(16, shape)
    x[0, 1, 37, 80] = value
    print("case ssim large", shape, value, flush=True)
    _check(x, y)


def test_identical_images_give_exactly_no_gradient():
    x, _ = _pair(17, STRIPS)
    print("case ssim identical", flush=True)
    loss, ssim, g = _gpu(x, x, 0.2)
    assert abs(loss) < 1e-6 * x.shape[0] and np.all(np.abs(ssim - 1.0) < 1e-6)
    assert np.all(g == 0.0)


@pytest.mark.parametrize("noise", [0.1, 0.02])
def test_no_further_from_64_bits_than_in_tiles(noise):
    """Six views together are taken in strips, each alone in tiles: the
    gradient's root mean square error is no larger (7e5 values of a view's
    rounding errors, which two draws give to well within 1 %)."""
    rng = np.random.default_rng(18)
    V, H, W = 6, 160, 300
    r, c = np.mgrid[0:H, 0:W]
    y = 0.5 + 0.45 * np.sin(r / 9.0 + rng.uniform(0, 6, (V, 3, 1, 1))) * np.cos(c / 13.0)
    x = np.clip(y + noise * rng.normal(size=y.shape), 0, 1).astype(np.float32)
    y = np.clip(y, 0, 1).astype(np.float32)
    print("case ssim error", noise, flush=True)
    strips = _gpu(x, y, 0.2)[2]
    tiles = np.concatenate([_gpu(x[k:k + 1], y[k:k + 1], 0.2)[2] for k in range(V)])
    ref = OS.loss_ssim(x.astype(np.float64), y.astype(np.float64), 0.2)[1]
    err = [np.sqrt(np.mean((g - ref) ** 2)) for g in (strips, tiles)]
    print("rms error, strips and tiles", err, "of", np.sqrt(np.mean(ref ** 2)))
    assert err[0] <= 1.01 * err[1]
