"""The dominated pixels per Gaussian, which the densification collects per
4,096 consecutive pixels before it adds them: the Gaussians above the
threshold, against counts on the host, for single pixels, around a chunk's
end, for chunks of as many Gaussians as pixels (the table's probes run out)
and for indices that stand for no Gaussian."""
import numpy as np
import pytest
import torch

import synth
from paper_2504_02437_amd import raster as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pixels,spread", [
    (1, 3), (4095, 40), (4096, 4096), (4097, 9000), (20000, 6000), (50001, 5)])
@pytest.mark.parametrize("sigma", [0, 1, 7])
def test_split_count_matches_the_host(pixels, spread, sigma):
    n = 9000
    w = synth.tiny_scene(85, n=n)
    rng = np.random.default_rng(pixels + sigma)
    dom = rng.integers(-1, spread, pixels).astype(np.int32)
    if pixels == 4096:
        dom = rng.permutation(n)[:pixels].astype(np.int32)   # all distinct
    dom[rng.integers(0, pixels, 3)] = 2 ** 30                # no Gaussian
    run = rng.integers(0, pixels)
    dom[run:run + 300] = 2                                   # across waves
    live = dom[(dom >= 0) & (dom < n)]
    want = int((np.bincount(live, minlength=n) > sigma).sum())
    p = R.ParamBuffer.from_gaussians(w.gaussians, capacity=2 * n)
    xi = torch.zeros(2 * n, 2, 3, device="cuda")
    n_split = torch.zeros(1, dtype=torch.int32, device="cuda")
    print("case dominant count", pixels, spread, sigma, flush=True)
    R.densify(p, p.zeros_like(), p.zeros_like(), torch.from_numpy(dom).cuda(),
              sigma, xi, n_split=n_split)
    torch.cuda.synchronize()
    assert int(n_split) == want and int(p.n_dev) == n + want
