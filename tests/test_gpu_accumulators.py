"""The compositing backward's per-Gaussian FP64 accumulators: the entry points
that pass through them (tiles below 32, 450 tiles and more) publish the same planar gradients as the direct adds, and leave the
accumulators clear."""
import numpy as np
import pytest

import synth
from gpu_helpers import (check_grads, check_screen_grads, gpu_backward_screen,
                         gpu_forward, masked_dL, oracle_backward,
                         oracle_forward)
from paper_2504_02437_amd import raster as R

pytestmark = pytest.mark.gpu


def _scene(views, n, W, H, degree=0):
    w = synth.tiny_scene(81, n=n, width=W, height=H, f=0.6 * W,
                         log_scale_mu=-3.5)
    w.gaussians = synth.with_sh(w.gaussians, 5, degree, 0.05)
    c = w.cameras[0]
    w.cameras = [synth.Camera(c.R, (c.t + np.array([0.04 * k, 0.0, 0.0])
                                    ).astype(np.float32), c.fx, c.fy, c.cx,
                              c.cy, W, H) for k in range(views)]
    return w


# All of these pass through the accumulators.
@pytest.mark.parametrize("views,W,H,tile,degree", [
    (1, 632, 632, 16, 0), (1, 608, 658, 16, 0), (2, 449, 449, 16, 2),
    (3, 401, 353, 8, 0), (1, 640, 640, 8, 1)])
def test_published_gradients_match_the_oracle(views, W, H, tile, degree):
    w = _scene(views, 1500, W, H, degree)
    print("case accumulators", views, W, H, tile, degree, flush=True)
    p64, proj, bins, fwd = oracle_forward(w, tile)
    params, rast = gpu_forward(w, tile)
    mask = fwd["flags"] == 0
    dL = masked_dL(np.random.default_rng(8), mask, (views, 3, H, W))
    ref, mag, b = oracle_backward(w, p64, proj, bins, dL, full=True)
    n = w.gaussians.n
    first = None
    for _ in range(2):   # the second call starts from cleared accumulators
        got, _, _ = gpu_backward_screen(
            rast, params, dL,
            check=lambda g: check_screen_grads(rast, g, b, n))
        check_grads(got, ref, n, mag=mag)
        first = got if first is None else first
    # Twice the same sums, up to the order of the FP32 adds within a tile.
    np.testing.assert_allclose(got, first, rtol=1e-3,
                               atol=1e-5 * np.abs(first).max())
