"""The projection of a single view forms the Gaussians' shapes itself, that of
several views reads them from a launch before: the same records, boxes, depths
and opacity logarithms bit for bit, at the ends of a workgroup's 256 Gaussians
and with shapes and positions that are culled."""
import numpy as np
import pytest
import torch

import synth
from gpu_helpers import gpu_forward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 255, 256, 257, 1000])
@pytest.mark.parametrize("full_box", [False, True])
def test_single_view_equals_the_first_of_two(n, full_box):
    w = synth.tiny_scene(87, n=n, width=61, height=47, f=50.0)
    g = w.gaussians
    if n > 8:
        g.quat[:, 1] = 0.0                    # no rotation: culled
        g.log_scale[0, 2] = np.nan
        g.mean[2, 3] = -1.0                   # behind the camera
        g.opacity_logit[..., 4] = -30.0       # never admitted
        g.mean[0, 5] = np.inf
    print("case project single", n, full_box, flush=True)
    _, one = gpu_forward(w, 16, full_box=full_box)
    w.cameras = [w.cameras[0], w.cameras[0]]
    _, two = gpu_forward(w, 16, full_box=full_box)
    t1, t2 = one.ws.tiles_touched()[0, :n], two.ws.tiles_touched()[0, :n]
    assert torch.equal(t1, t2)
    on = t1 > 0
    r1 = one.ws.records()[0, :n][on].view(torch.int32)
    r2 = two.ws.records()[0, :n][on].view(torch.int32)
    assert torch.equal(r1, r2)
    assert torch.equal(one.rgb[0], two.rgb[0])
    assert torch.equal(one.T[0], two.T[0]) and torch.equal(one.nlast[0], two.nlast[0])
