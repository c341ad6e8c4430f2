"""Chunk sizes of the tile binning (512, 1024 or 2048 Gaussians, by the grid
and the number of workgroups) and its key enumeration: keys and ranges against
the oracle, for chunk counts around the rule's 768 workgroups and for waves
whose Gaussians cover far more tiles than one span of the enumeration."""
import numpy as np
import pytest

import synth
from gpu_helpers import check_records, check_sort, gpu_forward, oracle_forward
from paper_2504_02437_amd import raster as R

pytestmark = pytest.mark.gpu


def _views(w, V):
    c = w.cameras[0]
    w.cameras = [synth.Camera(c.R, (c.t + np.array([0.03 * k, 0.0, 0.0])
                                    ).astype(np.float32), c.fx, c.fy, c.cx,
                              c.cy, c.width, c.height) for k in range(V)]
    return w


# capacity x views around 768 workgroups of 2048, 1024 and 512; the live
# Gaussians (2,500) end inside a chunk.
@pytest.mark.parametrize("W,H,tile,V,cap", [
    (320, 160, 16, 1, 2500),            # 200 tiles, chunks of 512
    (320, 160, 16, 2, 383 * 1024),      # 766 workgroups of 1024: 512
    (320, 160, 16, 2, 384 * 1024),      # 768: 1024
    (640, 480, 16, 1, 2500),            # 1,200 tiles, chunks of 512
    (640, 480, 16, 2, 384 * 1024),      # 1024
    (640, 480, 16, 2, 384 * 2048),      # 2048
    (1024, 1008, 16, 1, 3000),          # 4,032 tiles: 512
    (1040, 1024, 16, 1, 3000)])         # 4,160 tiles: 2048
def test_chunk_sizes(W, H, tile, V, cap):
    w = _views(synth.tiny_scene(83, n=2500, width=W, height=H, f=0.7 * W,
                                log_scale_mu=-3.0), V)
    print("case chunks", W, H, tile, V, cap, flush=True)
    p64, proj, bins, _ = oracle_forward(w, tile)
    params = R.ParamBuffer.from_gaussians(w.gaussians, capacity=cap)
    params, rast = gpu_forward(w, tile, params=params,
                               key_capacity=len(bins["vals"]) + 1024)
    n = w.gaussians.n
    rec = rast.ws.records
    rast.ws.records = lambda: rec()[:, :n]
    tt, rb = rast.ws.tiles_touched, rast.ws.render_box
    rast.ws.tiles_touched = lambda: tt()[:, :n]
    rast.ws.render_box = lambda: rb()[:, :n]
    check_records(rast, proj)
    check_sort(rast, bins)


# 150 Gaussians that cover most of 4,032 tiles, small ones between them: about
# 250,000 keys in one wave, and owners that span several masks.
def test_waves_of_very_large_gaussians():
    w = synth.tiny_scene(84, n=600, width=1024, height=1008, f=700.0,
                         log_scale_mu=-3.0)
    w.gaussians.log_scale[:, ::4] = 0.0
    print("case large", flush=True)
    p64, proj, bins, _ = oracle_forward(w, 16)
    assert len(bins["vals"]) > 300_000
    _, rast = gpu_forward(w, 16, key_capacity=len(bins["vals"]) + 1024)
    check_sort(rast, bins)
