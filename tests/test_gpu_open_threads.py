"""The launch shape that is picked when the caller leaves the threads open
gives the same images as every other."""
import pytest
import torch

import synth
from gpu_helpers import gpu_forward

pytestmark = pytest.mark.gpu


def _scene(n, W, H):
    w = synth.tiny_scene(81, n=n, width=W, height=H, f=0.6 * W,
                         log_scale_mu=-3.5)
    return w


# Tile grids at the edges of the rule for open threads: 2047, 2048, 8190 and
# 8192 tiles.
@pytest.mark.parametrize("tx,ty", [(89, 23), (64, 32), (91, 90), (128, 64)])
def test_open_threads_render_the_same_image(tx, ty):
    w = _scene(3000, 16 * tx - 5, 16 * ty - 3)
    print("case open threads", tx, ty, flush=True)
    _, base = gpu_forward(w, 16)
    assert (base.ws.tiles_x, base.ws.tiles_y) == (tx, ty)
    for threads in (64, 128, 256):
        _, r = gpu_forward(w, 16, threads=threads)
        assert torch.equal(r.rgb, base.rgb) and torch.equal(r.T, base.T)
        assert torch.equal(r.nlast, base.nlast)
