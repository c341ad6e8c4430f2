"""The nearest-mean searches at the sizes and shapes where their bounds, lists
and fallbacks change hands: exact neighbours and FP64 distances against the
oracle for maps below, at and above the list and group sizes, patches whose
reach holds more means than a list, equal distances, and means too far for the
FP32 bounds."""
import numpy as np
import pytest
import torch

import oracle
import oracle.mlp as OM
import synth
from paper_2504_02437_amd import raster as R

pytestmark = pytest.mark.gpu


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _check(means, cam, pts, centre_only, sample=None):
    """Both searches over the map `means` [3][n] (spare capacity behind it)."""
    n = means.shape[1]
    rng = np.random.default_rng(1)
    W, H = cam.width, cam.height
    img = rng.uniform(size=(3, H, W)).astype(np.float32)
    params = R.ParamBuffer(n + 40 * 9, n=n)
    params.data[0:3, :n] = _dev(means.astype(np.float32))
    params.data[0:3, n:] = 0.1           # spare slots are not in the map
    rgb = rng.uniform(size=(3, n)).astype(np.float32)
    params.data[11:14, :n] = _dev(rgb)
    per = 1 if centre_only else 9
    C = pts.shape[0] * per
    feats = torch.empty(C, 32, device="cuda")
    kidx = torch.empty(C, 8, dtype=torch.int32, device="cuda")
    kd = torch.empty(C, 8, device="cuda")
    cam_d = R.cameras_to_device([cam])
    R.knn_features(params, cam_d, W, H, _dev(img), _dev(pts), centre_only,
                   feats, kidx, kd)
    torch.cuda.synchronize()
    sel = np.arange(pts.shape[0]) if sample is None else np.asarray(sample)
    F, P = OM.features(cam, img, pts[sel], means.astype(np.float64),
                       rgb.astype(np.float64), centre_only)
    idx, dist = OM.knn(means.astype(np.float64), P)
    rows = (sel[:, None] * per + np.arange(per)).ravel()
    k = min(8, n)
    got = kidx.cpu().numpy()[rows]
    np.testing.assert_array_equal(got[:, :k], idx[:, :k])
    assert np.all(got[:, k:] == -1)
    np.testing.assert_allclose(kd.cpu().numpy()[rows][:, :k], dist[:, :k], rtol=1e-6)
    assert np.all(kd.cpu().numpy()[rows][:, k:] == 0)
    np.testing.assert_allclose(feats.cpu().numpy()[rows], F, rtol=1e-6, atol=1e-6)
    # The distance test: FP64 bits of the nearest squared distances.
    d2 = oracle.nearest(cam, pts, means.astype(np.float32), centre_only=centre_only,
                        nthreads=8)
    scratch = R.insert_distance(params, None, None, cam_d, W, H, _dev(img),
                                _dev(pts), 1e30, centre_only=centre_only)
    torch.cuda.synchronize()
    bits = scratch.cpu().numpy().view(np.uint64)
    inside = d2 >= 0
    np.testing.assert_array_equal(bits != np.uint64(0xFFFFFFFFFFFFFFFF), inside)
    np.testing.assert_array_equal(bits.view(np.float64)[inside], d2[inside])


def _camera(W=120, H=90, f=80.0):
    return synth.room_camera(W, H, f)


def _pts(rng, cam, K):
    return np.stack([rng.integers(1, cam.width - 1, K),
                     rng.integers(1, cam.height - 1, K),
                     1.0 / rng.uniform(1, 4, K)], 1).astype(np.float32)


@pytest.mark.parametrize("centre_only", [False, True])
@pytest.mark.parametrize("n", [1, 7, 8, 9, 17, 64, 65, 130, 1030, 5000])
def test_map_sizes(n, centre_only):
    rng = np.random.default_rng(n)
    print("case near size", n, centre_only, flush=True)
    cam = _camera()
    _check(rng.uniform(-2, 2, size=(3, n)).astype(np.float32), cam,
           _pts(rng, cam, 17), centre_only)


# A pixel of the small camera is 0.1 to 0.2 m wide: reach holds hundreds of
# the room's means (more than a list), and thousands of the dense cluster's
# (more than the larger list).
@pytest.mark.parametrize("centre_only", [False, True])
@pytest.mark.parametrize("cluster", [0, 30000])
def test_reach_beyond_the_lists(cluster, centre_only):
    rng = np.random.default_rng(5)
    print("case near reach", cluster, centre_only, flush=True)
    cam = _camera(40, 30, 20.0)
    means = synth.room_gaussians(rng, 40000).mean
    pts = _pts(rng, cam, 5)
    if cluster:
        R_, t = np.asarray(cam.R, np.float64), np.asarray(cam.t, np.float64)
        z = 1.0 / pts[2, 2]
        X = R_.T @ (np.array([(pts[2, 0] - cam.cx) / cam.fx * z,
                              (pts[2, 1] - cam.cy) / cam.fy * z, z]) - t)
        means = np.concatenate([means, (X[:, None] + rng.normal(
            0, 0.05, size=(3, cluster)))], 1)
    _check(means.astype(np.float32), cam, pts, centre_only)


@pytest.mark.parametrize("centre_only", [False, True])
def test_many_equal_means(centre_only):
    rng = np.random.default_rng(6)
    print("case near equal", centre_only, flush=True)
    cam = _camera()
    means = np.repeat(rng.uniform(-1, 1, size=(3, 3)), 200, axis=1)
    _check(means.astype(np.float32), cam, _pts(rng, cam, 4), centre_only)


@pytest.mark.parametrize("far", ["some", "all"])
def test_means_beyond_the_bounds(far):
    """Coordinates whose squares overflow FP32."""
    rng = np.random.default_rng(7)
    print("case near far", far, flush=True)
    cam = _camera()
    means = rng.uniform(-2, 2, size=(3, 700))
    if far == "all":
        means *= 1e22
    else:
        means[:, ::50] *= 1e25
        means[0, 3] = 2e19
    _check(means.astype(np.float32), cam, _pts(rng, cam, 6), False)


def test_many_patches():
    rng = np.random.default_rng(8)
    print("case near many", flush=True)
    cam = _camera(600, 400, 300.0)
    means = synth.room_gaussians(rng, 30000).mean
    _check(means, cam, _pts(rng, cam, 700), False,
           sample=[0, 15, 16, 333, 699])


@pytest.mark.parametrize("corner", [2, 6])
def test_sheared_camera_beyond_the_list(corner):
    """A rotation that is not orthonormal: the corners 2 and 6 of a patch are
    six times as far from its middle as 0 and 8, and the means around one of
    them, more than a list holds, are its neighbours."""
    rng = np.random.default_rng(9)
    print("case near sheared", corner, flush=True)
    shear = np.array([[1, 0, 0], [-0.9, 0.3, 0], [0, 0, 1]], np.float32)
    cam = synth.Camera(shear, np.zeros(3, np.float32), 20.0, 20.0, 20.0, 15.0,
                       40, 30)
    pts = np.array([[20, 15, 0.5]], np.float32)
    P = OM.features(cam, np.zeros((3, 30, 40), np.float32), pts,
                    np.zeros((3, 1)), np.zeros((3, 1)), False)[1]
    far = [np.linalg.norm(P[i] - P[4]) for i in (0, 2, 6, 8)]
    assert min(far[1:3]) > 5 * max(far[0], far[3])
    means = np.repeat(P[[4, corner]], 400, axis=0).T
    means = means + rng.normal(0, 1e-3, size=means.shape)
    _check(means.astype(np.float32), cam, pts, False)


@pytest.mark.parametrize("out", [50.0, 1000.0, 3e4])
@pytest.mark.parametrize("centre_only", [False, True])
def test_far_from_the_origin(out, centre_only):
    """Camera and map away from the world's origin: the same neighbours as
    the oracle's, and (in the second test) without every mean in reach."""
    rng = np.random.default_rng(11)
    print("case near far out", out, centre_only, flush=True)
    c = _camera(600, 400, 300.0)
    shift = np.array([out, -0.7 * out, 0.4 * out])
    t = (c.t - np.asarray(c.R, np.float64) @ shift).astype(np.float32)
    cam = synth.Camera(c.R, t, c.fx, c.fy, c.cx, c.cy, c.width, c.height)
    means = synth.room_gaussians(rng, 20000).mean + shift[:, None]
    _check(means.astype(np.float32), cam, _pts(rng, cam, 40), centre_only)


def test_bounds_are_as_tight_far_from_the_origin():
    """1 km out the neighbour search takes no more than three times as long as
    at the origin (every mean in reach: a hundred times)."""
    us = []
    for out in (0.0, 1000.0):
        rng = np.random.default_rng(12)
        print("case near far out time", out, flush=True)
        c = _camera(600, 400, 300.0)
        shift = np.full(3, out)
        t = (c.t - np.asarray(c.R, np.float64) @ shift).astype(np.float32)
        cam_d = R.cameras_to_device([synth.Camera(c.R, t, c.fx, c.fy, c.cx,
                                                  c.cy, c.width, c.height)])
        mean = synth.room_gaussians(rng, 200000).mean + shift[:, None]
        params = R.ParamBuffer(200000, n=200000)
        params.data[0:3] = _dev(mean.astype(np.float32))
        pts = _dev(_pts(rng, c, 96))
        img = torch.zeros(3, c.height, c.width, device="cuda")
        feats = torch.empty(96 * 9, 32, device="cuda")
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        for k in range(4):
            if k == 1:
                a.record()
            R.knn_features(params, cam_d, c.width, c.height, img, pts, False, feats)
        b.record()
        torch.cuda.synchronize()
        us.append(a.elapsed_time(b) / 3 * 1e3)
    print("us at 0 and 1000 m", us)
    assert us[1] <= 3 * us[0]
