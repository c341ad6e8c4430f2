"""Tile ranges of one view by a single workgroup (at most 1,024 tiles and 64
chunks of Gaussians) and by the two launches for more: keys and ranges against
the oracle around both lines, and the key count and overflow flag when the
keys do not fit."""
import pytest

import synth
from gpu_helpers import check_records, check_sort, gpu_forward, oracle_forward
from paper_2504_02437_amd import raster as R

pytestmark = pytest.mark.gpu


# 1, 6, 1,024 and 1,056 tiles; 64 and 65 chunks of 512 (by the capacity).
@pytest.mark.parametrize("W,H,n,cap", [
    (9, 7, 30, 30), (45, 29, 513, 513), (512, 512, 2000, 2000),
    (512, 528, 2000, 2000), (320, 240, 1500, 64 * 512),
    (320, 240, 1500, 64 * 512 + 1)])
def test_ranges_match_the_oracle(W, H, n, cap):
    w = synth.tiny_scene(89, n=n, width=W, height=H, f=0.7 * W,
                         log_scale_mu=-2.5)
    print("case small ranges", W, H, n, cap, flush=True)
    _, proj, bins, _ = oracle_forward(w, 16)
    params = R.ParamBuffer.from_gaussians(w.gaussians, capacity=cap)
    params, rast = gpu_forward(w, 16, params=params,
                               key_capacity=len(bins["vals"]) + 1024)
    rec, tt, rb = rast.ws.records, rast.ws.tiles_touched, rast.ws.render_box
    rast.ws.records = lambda: rec()[:, :n]
    rast.ws.tiles_touched = lambda: tt()[:, :n]
    rast.ws.render_box = lambda: rb()[:, :n]
    check_records(rast, proj)
    check_sort(rast, bins)


def test_overflow_is_reported():
    w = synth.tiny_scene(89, n=400, width=100, height=80, f=70.0,
                         log_scale_mu=-2.5)
    params = R.ParamBuffer.from_gaussians(w.gaussians)
    rast = R.Rasterizer(w.cameras, params.capacity, R.Settings(tile=16),
                        key_capacity=300, device="cuda")
    R.project_and_bin(rast.ws, params, rast.cams_dev, rast.settings)
    flags, keys = rast.status()
    assert flags != 0 and keys > 300
