"""The projection of many (view, Gaussian) pairs, which first drops those that
certainly touch no pixel (by capacity times views, so that the same Gaussians
take either form): tile counts of every pair, and records, boxes and images
bit for bit, for Gaussians of all sizes around every edge of the image, the
near plane and the camera's plane, and values that are not finite."""
import numpy as np
import pytest
import torch

import synth
from gpu_helpers import gpu_forward
from paper_2504_02437_amd import raster as R

pytestmark = pytest.mark.gpu


def _scene(seed, n, scale):
    w = synth.tiny_scene(seed, n=n, width=97, height=61, f=70.0)
    g, rng = w.gaussians, np.random.default_rng(seed)
    z = rng.choice([-1.0, 1.0], n, p=[0.2, 0.8]) * 10 ** rng.uniform(-2.5, 1.5, n)
    # On and around the edges of the frustum, and anywhere.
    edge = rng.choice([-1.0, 1.0, 0.0], n) * 97 / 140
    g.mean[0] = z * (edge + rng.normal(0, 0.3, n))
    g.mean[1] = z * (rng.choice([-1.0, 1.0, 0.0], n) * 61 / 140 + rng.normal(0, 0.3, n))
    g.mean[2] = z
    g.log_scale[:] = rng.normal(scale, 1.5, (3, n))
    g.mean[0, 3], g.mean[2, 4], g.log_scale[1, 5] = np.inf, np.nan, np.nan
    g.log_scale[0, 6], g.log_scale[2, 7] = 80.0, -80.0
    g.quat[:, 8] = 0.0
    c = w.cameras[0]
    a = 0.4
    turn = np.array([[np.cos(a), 0, np.sin(a)], [0, 1, 0],
                     [-np.sin(a), 0, np.cos(a)]], np.float32)
    w.cameras = [c, synth.Camera(turn, np.array([0.2, -0.1, 0.3], np.float32),
                                 c.fx, c.fy, 10.0, 80.0, c.width, c.height)]
    return w


@pytest.mark.parametrize("n,scale", [(1000, -4.0), (1025, -2.0), (5000, -6.0),
                                     (3000, 0.0)])
def test_same_pairs_as_one_by_one(n, scale):
    w = _scene(91 + n, n, scale)
    print("case project shared", n, scale, flush=True)
    out = []
    for cap in (n, 1 << 19):       # two views: 2^20 pairs
        params = R.ParamBuffer.from_gaussians(w.gaussians, capacity=cap)
        _, r = gpu_forward(w, 16, params=params, key_capacity=1 << 18)
        assert r.status()[0] == 0
        out.append(r)
    a, b = out
    ta, tb = a.ws.tiles_touched()[:, :n], b.ws.tiles_touched()[:, :n]
    assert torch.equal(ta, tb)
    on = ta > 0
    assert on.any() and not on.all()
    assert torch.equal(a.ws.records()[:, :n][on].view(torch.int32),
                       b.ws.records()[:, :n][on].view(torch.int32))
    assert torch.equal(a.ws.render_box()[:, :n][on], b.ws.render_box()[:, :n][on])
    assert torch.equal(a.T, b.T) and torch.equal(a.nlast, b.nlast)


@pytest.mark.parametrize("near", [-30.0, 0.0, float("nan")])
def test_near_planes_behind_the_camera(near):
    """A near plane that lets Gaussians behind the camera through (or, not a
    number, nothing): the same pairs in either form."""
    n = 3000
    w = _scene(17, n, -3.0)
    for c in w.cameras:
        c.near = near
    print("case project shared near", near, flush=True)
    tiles = []
    for cap in (n, 1 << 19):
        params = R.ParamBuffer.from_gaussians(w.gaussians, capacity=cap)
        _, r = gpu_forward(w, 16, params=params, key_capacity=1 << 18)
        assert r.status()[0] == 0
        tiles.append(r.ws.tiles_touched()[:, :n].clone())
    behind = torch.from_numpy(w.gaussians.mean[2] < 0).cuda()
    assert bool((tiles[0][0][behind] > 0).any()) == (near < 0)
    assert torch.equal(tiles[0], tiles[1])
