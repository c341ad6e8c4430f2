"""The compositing kernels that take few tiles in 8x8 blocks, four entries of
a list side by side: images, transmittance and last contributor bit for bit as
from one workgroup per tile, gradients within the oracle's bounds."""
import numpy as np
import pytest
import torch

import synth
from gpu_helpers import (check_grads, check_screen_grads, gpu_backward_screen,
                         gpu_forward, masked_dL, oracle_backward,
                         oracle_forward)
from paper_2504_02437_amd import raster as R

pytestmark = pytest.mark.gpu


def _scene(W, H, n, views=1, scale=-2.5, seed=83):
    w = synth.tiny_scene(seed, n=n, width=W, height=H, f=0.8 * W,
                         log_scale_mu=scale)
    w.gaussians.opacity_logit[..., ::7] = 9.0      # above alpha_max
    c = w.cameras[0]
    w.cameras = [synth.Camera(c.R, (c.t + np.array([0.05 * k, 0.0, 0.0])
                                    ).astype(np.float32), c.fx, c.fy, c.cx,
                              c.cy, W, H) for k in range(views)]
    return w


BG = (0.2, 0.5, 0.1)
# Ragged images, a single block, lists past one batch of 256, several views,
# and both sides of the rule's lines: 1,300 blocks (3,000 backward at tile 8).
FORWARD = [(7, 5, 40, 1, 16), (33, 29, 300, 1, 16), (50, 41, 1500, 2, 16),
           (161, 119, 900, 1, 16), (40, 27, 700, 3, 8), (9, 8, 30, 1, 8),
           (320, 256, 500, 1, 16), (320, 260, 500, 1, 16),
           (304, 400, 500, 1, 16), (320, 255, 500, 1, 8),
           (320, 265, 500, 1, 8)]


@pytest.mark.parametrize("W,H,n,views,tile", FORWARD)
@pytest.mark.parametrize("bg", [(0.0, 0.0, 0.0), BG])
def test_same_decisions_as_one_workgroup_per_tile(W, H, n, views, tile, bg):
    w = _scene(W, H, n, views)
    print("case split forward", W, H, n, views, tile, bg, flush=True)
    _, a = gpu_forward(w, tile, bg=bg)
    _, b = gpu_forward(w, tile, bg=bg, threads=64 if tile == 8 else 256)
    assert torch.equal(a.T, b.T) and torch.equal(a.nlast, b.nlast)
    assert torch.equal(a.rgb, b.rgb)


# 320 and 1,260 blocks, 1,300 (one workgroup per tile); tile 8 below and at
# its line.
@pytest.mark.parametrize("W,H,n,views,tile", [
    (33, 29, 300, 1, 16), (50, 41, 1500, 2, 16), (160, 120, 900, 1, 16),
    (240, 336, 700, 1, 16), (320, 260, 700, 1, 16), (40, 27, 700, 3, 8),
    (160, 180, 700, 1, 8), (400, 480, 700, 1, 8)])
@pytest.mark.parametrize("bg", [(0.0, 0.0, 0.0), BG])
def test_gradients_match_the_oracle(W, H, n, views, tile, bg):
    w = _scene(W, H, n, views)
    print("case split backward", W, H, n, views, tile, bg, flush=True)
    p64, proj, bins, fwd = oracle_forward(w, tile, bg)
    params, rast = gpu_forward(w, tile, bg=bg)
    dL = masked_dL(np.random.default_rng(8), fwd["flags"] == 0, (views, 3, H, W))
    ref, mag, b = oracle_backward(w, p64, proj, bins, dL, bg, full=True)
    n = w.gaussians.n
    got, _, _ = gpu_backward_screen(
        rast, params, dL, check=lambda g: check_screen_grads(rast, g, b, n))
    check_grads(got, ref, n, mag=mag)


@pytest.mark.parametrize("W,H,views,tile", [(33, 29, 2, 16), (320, 257, 1, 16),
                                            (320, 256, 1, 16), (45, 70, 1, 8),
                                            (640, 400, 1, 16), (330, 300, 3, 16)])
def test_fused_l1_matches_the_separate_loss(W, H, views, tile):
    """Loss and squared errors (a slot per block or tile), which the fused call
    sums in a fixed order, by a launch of its own or beside the accumulators'
    pass: the same twice."""
    w = _scene(W, H, 400, views)
    params, rast = gpu_forward(w, tile, bg=BG)
    rng = np.random.default_rng(9)
    tgt = torch.from_numpy(rng.uniform(size=(views, 3, H, W)).astype(np.float32)).cuda()
    print("case split l1", W, H, views, tile, flush=True)
    f64 = dict(dtype=torch.float64, device="cuda")
    ref, refsq = torch.zeros(1, **f64), torch.zeros(views, **f64)
    dL = torch.empty_like(rast.rgb)
    R.loss_l1(rast.rgb, tgt, 0.75, dL, ref, refsq)
    ga = params.zeros_like()
    R.render_bwd_pixels(rast.ws, params, rast.settings, dL, rast.T, rast.nlast, ga)
    R.project_bwd(rast.ws, params, rast.cams_dev, ga)
    out = []
    for _ in range(2):
        grad, loss, sq = params.zeros_like(), torch.zeros(1, **f64), torch.zeros(views, **f64)
        rast.backward_l1(params, tgt, 0.75, grad, loss, sq)
        torch.cuda.synchronize()
        out.append((float(loss), sq.cpu().numpy()))
    assert out[0][0] == out[1][0] and np.array_equal(out[0][1], out[1][1])
    assert out[0][0] == pytest.approx(float(ref), rel=1e-6)
    np.testing.assert_allclose(out[0][1], refsq.cpu().numpy(), rtol=1e-12)
    scale = ga.data.abs().amax(dim=1, keepdim=True)
    assert ((grad.data - ga.data).abs() <= 1e-5 * scale + 1e-12).all()
