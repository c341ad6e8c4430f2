"""The work that a user of this framework has it do, as cases that can be
timed and compared: single-view training steps, keyframe-window iterations,
the colour loss, keyframe insertion, densification, the optimiser and the
training of the learned initialisation, over the sizes of this repository's
workloads (160x120 with 10k Gaussians up to a 10-view 1200x680 window over
300k Gaussians) and the ragged sizes between them."""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2504_02437_amd import raster as R
from paper_2504_02437_amd.init_mlp import InitMLP, init_weights

DEV = "cuda"
ALPHA_MIN = float(np.float32(1.0) / np.float32(255.0))
T_MIN = float(np.float32(1e-4))
ALPHA_MAX = float(np.float32(0.99))
LAM_SSIM = 0.2


# ---- the cases -------------------------------------------------------------

def _view(name, width, height, f, n, views=1, tile=16, sh=0, bg=False):
    return dict(name=name, kind="step", width=width, height=height, f=f, n=n,
                views=views, tile=tile, sh=sh, bg=bg)


def listed():
    return [
        # Smallest scene: one 160x120 view of 10k Gaussians, default settings,
        # forward and backward of the L1 term (launch and latency bound).
        _view("step-160x120-10k", 160, 120, 128.0, 10_000),
        # One keyframe of a small mapping run (the 320x240 mapper workload),
        # with a background colour.
        _view("step-320x240-30k-bg", 320, 240, 260.0, 30_000, bg=True),
        # The per-keyframe path at full size, default settings.
        _view("step-1200x680-300k", 1200, 680, 600.0, 300_000),
        # Ragged sizes, several views, degree-3 view-dependent colour, tile 32.
        _view("step-5x517x389-61k-sh3", 517, 389, 430.0, 61_003, views=5,
              tile=32, sh=3),
        # The keyframe window as the library's graph (planar regulariser, no
        # optimiser step): the 640x480 window at the default settings ...
        dict(name="window-10x640x480-150k", kind="window", width=640,
             height=480, f=525.0, n=150_000, views=10, tile=16),
        # ... and the headline window at the autotuned launch shape.
        dict(name="window-10x1200x680-300k", kind="window", width=1200,
             height=680, f=600.0, n=300_000, views=10, tile=32),
        # Colour loss (L1 + SSIM) of the whole window, and of one small ragged
        # image.
        dict(name="colour-10x1200x680", kind="colour", width=1200, height=680,
             views=10),
        dict(name="colour-1x377x251", kind="colour", width=377, height=251,
             views=1),
        # Clarity-enhancing densification of one keyframe (dominant render,
        # count, split).
        dict(name="densify-1200x680-300k", kind="densify", width=1200,
             height=680, f=600.0, n=300_000),
        # Keyframe insertion by the distance test: 96 patches of 3x3
        # candidates against the whole map.
        dict(name="distance-96x9-300k", kind="distance", width=1200,
             height=680, f=600.0, n=300_000, patches=96),
        # Learned insertion: neighbour features, network, insertion.
        dict(name="learned-96x9-300k", kind="learned", width=1200, height=680,
             f=600.0, n=300_000, patches=96),
        # One training step of the learned initialisation (its batch size).
        dict(name="mlp-train-8192", kind="mlp", rows=8192),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _image(rng, lo, hi):
    w = _log(rng, lo, hi)
    return w, max(8, int(round(w * rng.uniform(0.55, 0.8))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "window", "window", "colour",
                       "densify", "distance", "learned", "mlp"])
    if kind == "colour":
        w, h = _image(rng, 64, 1200)
        return dict(kind=kind, width=w, height=h, views=rng.randint(1, 10))
    if kind == "mlp":
        return dict(kind=kind, rows=_log(rng, 500, 65_536))
    w, h = _image(rng, 150, 1200)
    f = round(w * rng.uniform(0.5, 0.85), 2)
    # Maps as dense per pixel as the repository's scenes (0.3 .. 0.6).
    n = max(1000, int(w * h * rng.uniform(0.25, 0.6)))
    n = min(n, 300_000)
    if kind == "step":
        return dict(kind=kind, width=w, height=h, f=f, n=n,
                    views=min(rng.choice([1, 1, 1, 2, 3, 5]),
                              max(1, 1_200_000 // (w * h))),
                    tile=rng.choice([16, 16, 32, 8 if w < 400 else 16]),
                    sh=rng.choice([0, 0, 0, 1, 2, 3]),
                    bg=rng.random() < 0.25)
    if kind == "window":
        tile = rng.choice([16, 32])
        most = max(1, (3_000_000 if tile == 16 else 8_000_000) // (w * h))
        return dict(kind=kind, width=w, height=h, f=f, n=n,
                    views=min(rng.randint(2, 10), most), tile=tile)
    if kind == "densify":
        return dict(kind=kind, width=w, height=h, f=f, n=n)
    return dict(kind=kind, width=w, height=h, f=f,
                n=_log(rng, 5_000, 300_000), patches=rng.randint(8, 192))


# ---- inputs ----------------------------------------------------------------

ROOM_LO, ROOM_HI = (-3.0, -1.5, -2.5), (3.0, 1.5, 2.5)


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 7919 + 17)


def _room(g, n, sh):
    """Gaussian rows [14 + sh rows][n]: 80% on the walls of a room (2 cm
    noise), the rest inside it; scales around 5 cm, opacities around 1/2."""
    U = lambda *s: torch.rand(*s, device=DEV, generator=g)
    N = lambda *s: torch.randn(*s, device=DEV, generator=g)
    lo = torch.tensor(ROOM_LO, device=DEV)
    hi = torch.tensor(ROOM_HI, device=DEV)
    ext = hi - lo
    pts = lo + U(n, 3) * ext
    area = torch.stack([ext[1] * ext[2], ext[0] * ext[2], ext[0] * ext[1]])
    axis = torch.multinomial(area, n, replacement=True, generator=g)
    side = torch.where(U(n) < 0.5, lo[axis], hi[axis])
    on_wall = U(n) < 0.8
    rows = torch.arange(n, device=DEV)
    pts[rows, axis] = torch.where(on_wall, side + 0.02 * N(n), pts[rows, axis])
    q = N(4, n)
    out = [pts.T, -3.0 + 0.5 * N(3, n), q / q.norm(dim=0, keepdim=True),
           N(1, n), U(3, n)]
    if sh:
        out.append(0.1 * N(R.sh_rows(sh), n))
    return torch.cat(out, 0).float().contiguous()


def _cameras(seed, views, width, height, f):
    """A keyframe walk: 5 cm and 3 degrees per step."""
    rng = np.random.default_rng([11, int(seed)])
    pos, yaw, pitch = np.array([0.0, 0.0, -0.5]), 0.0, 0.0
    yaw = rng.uniform(-0.3, 0.3)
    cams = []
    for _ in range(views):
        cy, sy, cp, sp = math.cos(yaw), math.sin(yaw), math.cos(pitch), math.sin(pitch)
        Rm = np.array([[cy, 0, -sy], [sy * sp, cp, cy * sp],
                       [sy * cp, -sp, cy * cp]])
        cams.append(SimpleNamespace(
            R=Rm.astype(np.float32), t=(-(Rm @ pos)).astype(np.float32),
            fx=float(f), fy=float(f), cx=(width - 1) / 2.0,
            cy=(height - 1) / 2.0, width=width, height=height, near=0.2))
        yaw += math.radians(3.0) * rng.uniform(0.5, 1.0)
        pitch += math.radians(1.0) * rng.uniform(-1.0, 1.0)
        pos = pos + 0.05 * rng.normal(size=3) / math.sqrt(3.0)
    return cams


def _params(data, spare=0):
    n = data.shape[1]
    sh = {14: 0, 23: 1, 38: 2, 59: 3}[data.shape[0]]
    if spare:
        data = torch.cat([data, torch.zeros(data.shape[0], spare, device=DEV)], 1)
    return R.ParamBuffer(n + spare, DEV, n, data.contiguous(), sh_degree=sh)


def _settings(case):
    # Tile 16 is the default; 32 takes the autotuner's batch and threads.
    bg = (0.2, 0.3, 0.4) if case.get("bg") else (0.0, 0.0, 0.0)
    if case["tile"] == 32:
        return R.Settings(tile=32, lds_batch=256, block_threads=256, bg=bg)
    return R.Settings(tile=case["tile"], bg=bg)


def _scene(case, seed):
    g = _gen(seed)
    data = _room(g, case["n"], case.get("sh", 0))
    V, W, H = case.get("views", 1), case["width"], case["height"]
    cams = _cameras(seed, V, W, H, case["f"])
    target = torch.rand(V, 3, H, W, device=DEV, generator=g)
    return g, data, cams, target


def _keyframe(g, case):
    """Patch centres (u, v, inverse depth) and the keyframe's image."""
    W, H, K = case["width"], case["height"], case["patches"]
    U = lambda *s: torch.rand(*s, device=DEV, generator=g)
    pts = torch.stack([(1 + U(K) * (W - 2)).floor(), (1 + U(K) * (H - 2)).floor(),
                       1.0 / (1.0 + 4.0 * U(K))], 1).float().contiguous()
    return pts, torch.rand(3, H, W, device=DEV, generator=g)


def prepare(case, seed):
    kind = case["kind"]
    s = SimpleNamespace(kind=kind, case=case)
    if kind in ("step", "window", "densify"):
        g, data, cams, s.target = _scene(case, seed)
        # Densification appends children: room for them.
        s.params = _params(data, case["n"] // 4 if kind == "densify" else 0)
        s.rast = R.Rasterizer(cams, s.params.capacity,
                              _settings({"tile": 16, **case}), device=DEV)
        s.rast.fit_key_capacity(s.params)
        s.grad = s.params.zeros_like()
        s.loss = torch.zeros(1, dtype=torch.float64, device=DEV)
        if kind == "window":
            st = torch.cuda.Stream()
            st.wait_stream(torch.cuda.current_stream())
            s.graph = R.WindowGraph(s.rast, s.params, s.grad, s.target, s.loss,
                                    lam_reg=1.0, stream=st)
            torch.cuda.current_stream().wait_stream(st)
        if kind == "densify":
            cap = s.params.capacity
            s.data0, s.n0 = s.params.data.clone(), s.params.n_dev.clone()
            s.m, s.v = s.params.zeros_like(), s.params.zeros_like()
            s.xi = torch.randn(cap, 2, 3, device=DEV, generator=g)
            s.scratch = R.densify_scratch(cap, DEV)
            s.n_split = torch.zeros(1, dtype=torch.int32, device=DEV)
            s.sigma = 24
    elif kind == "colour":
        g = _gen(seed)
        shape = (case["views"], 3, case["height"], case["width"])
        # A target with structure and a render that follows it, as in mapping.
        base = torch.nn.functional.interpolate(
            torch.rand(shape[0], 3, 2 + shape[2] // 9, 2 + shape[3] // 9,
                       device=DEV, generator=g), size=shape[2:],
            mode="bilinear", align_corners=False)
        noise = lambda a: a * torch.randn(shape, device=DEV, generator=g)
        s.target = (base + noise(0.05)).clamp(0, 1).contiguous()
        s.rgb = (base + noise(0.1)).clamp(0, 1).contiguous()
        s.dL = torch.empty(shape, device=DEV)
        s.loss = torch.zeros(1, dtype=torch.float64, device=DEV)
        s.scratch = R.ssim_scratch(s.rgb)
    elif kind in ("distance", "learned"):
        g, data, cams, _ = _scene(case, seed)
        s.params = _params(data, 9 * case["patches"])
        s.n0 = s.params.n_dev.clone()
        s.m, s.v = s.params.zeros_like(), s.params.zeros_like()
        s.cam = R.cameras_to_device(cams[:1], DEV)
        s.pts, s.img = _keyframe(g, case)
        C = 9 * case["patches"]
        s.n_ins = torch.zeros(1, dtype=torch.int32, device=DEV)
        if kind == "distance":
            s.scratch = torch.empty(C, dtype=torch.int64, device=DEV)
        else:
            s.T = torch.rand(case["height"], case["width"], device=DEV, generator=g)
            s.feats = torch.empty(C, 32, device=DEV)
            s.idx = torch.empty(C, 8, dtype=torch.int32, device=DEV)
            s.mlp = InitMLP.load(device=DEV)
    elif kind == "mlp":
        g = _gen(seed)
        M = case["rows"]
        s.x = torch.rand(M, 32, device=DEV, generator=g)
        s.t = torch.randn(M, 7, device=DEV, generator=g)
        # Some way into training: moments of the gradient's size.
        s.net = InitMLP(init_weights(int(seed) % 2 ** 31), device=DEV)
        s.net.m.copy_(1e-3 * torch.randn(s.net.m.shape, device=DEV, generator=g))
        s.net.v.fill_(1e-4)
        s.net.step = 200
    else:
        raise ValueError(kind)
    return s


# ---- one pass --------------------------------------------------------------

def run(s):
    c = s.case
    if s.kind == "step":
        s.grad.data.zero_()
        s.loss.zero_()
        rgb, T, nlast = s.rast.forward(s.params)
        s.rast.backward_l1(s.params, s.target, 1.0, s.grad, s.loss)
        # The loss in single precision, as a training log keeps it.
        return {"rgb": rgb, "T": T, "nlast": nlast, "grad": s.grad.data,
                "loss": s.loss.float()}
    if s.kind == "window":
        s.graph.run()
        return {"rgb": s.rast.rgb, "T": s.rast.T, "nlast": s.rast.nlast,
                "grad": s.grad.data, "loss": s.loss.float()}
    if s.kind == "colour":
        s.loss.zero_()
        R.loss_colour(s.rgb, s.target, 1.0 - LAM_SSIM, LAM_SSIM, s.dL, s.loss,
                      scratch=s.scratch)
        return {"dL": s.dL, "loss": s.loss.float()}
    if s.kind == "densify":
        # The map as it was before the pass.
        s.params.data.copy_(s.data0)
        s.params.n_dev.copy_(s.n0)
        dom = s.rast.forward_dominant(s.params)
        R.densify(s.params, s.m, s.v, dom, s.sigma, s.xi, scratch=s.scratch,
                  n_split=s.n_split)
        return {"rgb": s.rast.rgb, "T": s.rast.T, "dom": dom,
                "data": s.params.data, "n_split": s.n_split}
    if s.kind == "distance":
        s.params.n_dev.copy_(s.n0)
        R.insert_distance(s.params, s.m, s.v, s.cam, c["width"], c["height"],
                          s.img, s.pts, 0.02, scratch=s.scratch,
                          n_inserted_dev=s.n_ins)
        return {"nearest2": s.scratch, "data": s.params.data, "n_ins": s.n_ins}
    if s.kind == "learned":
        s.params.n_dev.copy_(s.n0)
        R.knn_features(s.params, s.cam, c["width"], c["height"], s.img, s.pts,
                       False, s.feats, s.idx)
        out = s.mlp.predict(s.feats)
        R.insert_gaussians(s.params, s.m, s.v, s.cam, c["width"], c["height"],
                           s.img, s.T, s.pts, 0.9, False, out, s.n_ins)
        return {"feats": s.feats, "idx": s.idx, "init": out,
                "data": s.params.data, "n_ins": s.n_ins}
    loss = s.net.train_step(s.x, s.t)
    return {"w": s.net.w, "g": s.net.g, "m": s.net.m, "loss": loss.float()}


# ---- what a pass cannot do without -----------------------------------------

# Contributing (pixel, Gaussian) pairs per pixel of these scenes.
PAIRS = 85


def work(case):
    kind = case["kind"]
    if kind == "colour":
        px = 3 * case["views"] * case["width"] * case["height"]
        return {"bytes": 12.0 * px, "flops": 2.0 * 190 * px}
    if kind == "mlp":
        M = case["rows"]
        return {"bytes": 4.0 * M * (32 + 7) + 6727 * 4 * 7.0,
                "flops": 3 * 2.0 * M * (32 * 64 + 64 * 64 + 64 * 7)}
    n, px = case["n"], case["width"] * case["height"]
    if kind in ("distance", "learned"):
        C = 9 * case["patches"]
        return {"bytes": 12.0 * n + 4.0 * C * (14 if kind == "distance" else 46),
                "flops": 8.0 * n * C}
    V = case.get("views", 1)
    rows = 14 + R.sh_rows(case.get("sh", 0))
    if kind == "densify":
        return {"bytes": 4.0 * rows * n + 20.0 * px, "flops": 20.0 * PAIRS * px}
    # Parameters read, gradients written, image / T / n_last written, target
    # read.
    return {"bytes": 8.0 * rows * n + 32.0 * V * px,
            "flops": 64.0 * PAIRS * V * px}


# ---- the same in 64 bits ---------------------------------------------------

def _project64(data, cam):
    """Screen-space quantities of every Gaussian in one view (64 bits,
    differentiable): px, py, conic A, B, C, depth, and the box radius."""
    d = lambda a: torch.as_tensor(np.asarray(a, np.float32).astype(np.float64), device=DEV)
    f32 = lambda v: float(np.float32(v))
    Wm, t = d(cam.R), d(cam.t)
    fx, fy, cx, cy = f32(cam.fx), f32(cam.fy), f32(cam.cx), f32(cam.cy)
    mean, sc, q = data[0:3], data[3:6].exp(), data[6:10]
    w, x, y, z = q / q.norm(dim=0, keepdim=True)
    Rm = torch.stack([
        torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)]),
        torch.stack([2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)]),
        torch.stack([2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)])])
    M = Rm * sc[None]
    tc = Wm @ mean + t[:, None]
    live = tc[2].detach() > f32(cam.near)
    tz = torch.where(live, tc[2], torch.ones_like(tc[2]))
    lx, ly = 1.3 * cam.width / (2 * fx), 1.3 * cam.height / (2 * fy)
    xc = (tc[0] / tz).clamp(-lx, lx) * tz
    yc = (tc[1] / tz).clamp(-ly, ly) * tz
    J0 = (fx / tz)[None] * Wm[0][:, None] - (fx * xc / tz ** 2)[None] * Wm[2][:, None]
    J1 = (fy / tz)[None] * Wm[1][:, None] - (fy * yc / tz ** 2)[None] * Wm[2][:, None]
    u0 = (J0[:, None] * M).sum(0)
    u1 = (J1[:, None] * M).sum(0)
    a = (u0 * u0).sum(0) + 0.3
    b = (u0 * u1).sum(0)
    c = (u1 * u1).sum(0) + 0.3
    det = a * c - b * b
    px, py = fx * tc[0] / tz + cx, fy * tc[1] / tz + cy
    with torch.no_grad():
        mid = 0.5 * (a + c)
        rad = (3.0 * (mid + (mid * mid - det).clamp_min(0.1).sqrt()).sqrt()).ceil()
        box = torch.stack([(px - rad).ceil().clamp_min(0),
                           (px + rad).floor().clamp_max(cam.width - 1),
                           (py - rad).ceil().clamp_min(0),
                           (py + rad).floor().clamp_max(cam.height - 1)])
        live = live & (box[0] <= box[1]) & (box[2] <= box[3])
        depth = tc[2].float()
    return torch.stack([px, py, c / det, -b / det, a / det]), depth, box, live


def _sh64(data, cam, degree):
    """Colour of every Gaussian in one view."""
    rgb = data[11:14]
    if not degree:
        return rgb
    Rm = torch.as_tensor(np.asarray(cam.R, np.float64), device=DEV)
    t = torch.as_tensor(np.asarray(cam.t, np.float64), device=DEV)
    v = data[0:3] + (Rm.T @ t)[:, None]
    x, y, z = v / v.norm(dim=0, keepdim=True)
    pi = math.pi
    c1 = math.sqrt(3 / (4 * pi))
    Y = [-c1 * y, c1 * z, -c1 * x]
    if degree >= 2:
        a, b, c = math.sqrt(15 / pi) / 2, math.sqrt(5 / pi) / 4, math.sqrt(15 / pi) / 4
        Y += [a * x * y, -a * y * z, b * (2 * z * z - x * x - y * y),
              -a * x * z, c * (x * x - y * y)]
    if degree >= 3:
        a, b = math.sqrt(35 / (2 * pi)) / 4, math.sqrt(105 / pi) / 2
        c, d, e = math.sqrt(21 / (2 * pi)) / 4, math.sqrt(7 / pi) / 4, math.sqrt(105 / pi) / 4
        Y += [-a * y * (3 * x * x - y * y), b * x * y * z,
              -c * y * (4 * z * z - x * x - y * y),
              d * z * (2 * z * z - 3 * x * x - 3 * y * y),
              -c * x * (4 * z * z - x * x - y * y), e * z * (x * x - y * y),
              -a * x * (x * x - 3 * y * y)]
    co = data[14:].reshape(len(Y), 3, -1)
    return (rgb + (torch.stack(Y)[:, None] * co).sum(0)).clamp_min(0)


def _composite64(rec, col, op, depth, box, live, bg, W, H, target=None,
                 lam=0.0, edge=64):
    """Image and transmittance of one view, square by square; with a target
    also the gradient of lam * mean |image - target| with respect to rec, op
    and col."""
    rgb = torch.zeros(3, H, W, dtype=torch.float64, device=DEV)
    T = torch.ones(H, W, dtype=torch.float64, device=DEV)
    grads = [torch.zeros_like(v) for v in (rec, col, op)] if target is not None else None
    order = torch.argsort(depth, stable=True)
    order = order[live[order]]
    bx = box[:, order]
    bgv = torch.tensor(bg, dtype=torch.float32, device=DEV).double()
    for v0 in range(0, H, edge):
        for u0 in range(0, W, edge):
            u1, v1 = min(W, u0 + edge), min(H, v0 + edge)
            meets = (bx[0] < u1) & (bx[1] >= u0) & (bx[2] < v1) & (bx[3] >= v0)
            ids = order[meets]
            uu = torch.arange(u0, u1, device=DEV, dtype=torch.float64)
            vv = torch.arange(v0, v1, device=DEV, dtype=torch.float64)
            with torch.enable_grad():
                leaf = [v[..., ids].detach().requires_grad_(target is not None)
                        for v in (rec, col, op)]
                r, cl, o = leaf
                b = box[:, ids]
                dx = r[0][:, None] - uu[None]
                dy = r[1][:, None] - vv[None]
                inx = (uu[None] >= b[0][:, None]) & (uu[None] <= b[1][:, None])
                iny = (vv[None] >= b[2][:, None]) & (vv[None] <= b[3][:, None])
                e = (-0.5 * (r[2][:, None] * dx * dx)[:, None, :]
                     - 0.5 * (r[4][:, None] * dy * dy)[:, :, None]
                     - (r[3][:, None] * dy)[:, :, None] * dx[:, None, :])
                al = (o[:, None, None] * e.exp()).clamp_max(ALPHA_MAX)
                ok = inx[:, None, :] & iny[:, :, None] & (al.detach() >= ALPHA_MIN)
                al = torch.where(ok, al, torch.zeros_like(al))
                lg = torch.log1p(-al)
                cum = lg.cumsum(0)
                con = ok & (cum.detach().exp() >= T_MIN)
                lg = torch.where(con, lg, torch.zeros_like(lg))
                w = torch.where(con, al, torch.zeros_like(al)) * (lg.cumsum(0) - lg).exp()
                Tf = lg.sum(0).exp()
                img = (cl @ w.reshape(w.shape[0], -1)).reshape(3, *Tf.shape)
                img = img + bgv[:, None, None] * Tf
                rgb[:, v0:v1, u0:u1] = img.detach()
                T[v0:v1, u0:u1] = Tf.detach()
                if target is not None and ids.numel():
                    d = lam * torch.sign(img.detach() - target[:, v0:v1, u0:u1])
                    for acc, gr in zip(grads, torch.autograd.grad(img, leaf, d)):
                        acc[..., ids] += gr
    return rgb, T, grads


def _exact_render(case, seed, with_grad):
    _, data32, cams, target = _scene(case, seed)
    bg = (0.2, 0.3, 0.4) if case.get("bg") else (0.0, 0.0, 0.0)
    W, H = case["width"], case["height"]
    data = data32.double().requires_grad_(with_grad)
    total = torch.zeros_like(data)
    rgbs, Ts, loss = [], [], 0.0
    for k, cam in enumerate(cams):
        with torch.set_grad_enabled(with_grad):
            rec, depth, box, live = _project64(data, cam)
            col = _sh64(data, cam, case.get("sh", 0))
            op = torch.sigmoid(data[10])
        tgt = target[k].double()
        scale = 1.0 / (3 * H * W)
        rgb, T, gr = _composite64(rec.detach(), col.detach(), op.detach(),
                                  depth, box, live, bg, W, H,
                                  tgt if with_grad else None, scale)
        rgbs.append(rgb)
        Ts.append(T)
        if with_grad:
            total += torch.autograd.grad([rec, col, op], data, gr)[0]
            loss += float((rgb - tgt).abs().sum()) * scale
    return torch.stack(rgbs), torch.stack(Ts), total, loss


def _exact_colour(case, seed):
    s = prepare(case, seed)
    H, W = case["height"], case["width"]
    g = torch.exp(-(torch.arange(11, device=DEV, dtype=torch.float64) - 5) ** 2 / 4.5)
    w = g / g.sum()

    def win(x):
        p = torch.nn.functional.pad(x, (5, 5, 5, 5))
        h = sum(w[i] * p[..., i:i + W] for i in range(11))
        return sum(w[i] * h[..., i:i + H, :] for i in range(11))

    dL, loss = torch.empty(s.rgb.shape, dtype=torch.float64, device=DEV), 0.0
    for k in range(case["views"]):
        x = s.rgb[k].double().requires_grad_(True)
        y = s.target[k].double()
        mx, my = win(x), win(y)
        cov = win(x * y) - mx * my
        var = win(x * x) - mx * mx + win(y * y) - my * my
        c1, c2 = 0.01 ** 2, 0.03 ** 2
        S = ((2 * mx * my + c1) * (2 * cov + c2)
             / ((mx * mx + my * my + c1) * (var + c2)))
        l = (1 - LAM_SSIM) * (x - y).abs().mean() + LAM_SSIM * (1 - S.mean())
        dL[k] = torch.autograd.grad(l, x)[0]
        loss += float(l)
    return {"dL": dL, "loss": torch.tensor([loss], dtype=torch.float64)}


def _candidates64(s, case):
    cam = _cameras(s.seed, 1, case["width"], case["height"], case["f"])[0]
    off = torch.arange(9, device=DEV)
    p = s.pts.double()
    u = (p[:, 0:1] + (off % 3 - 1)).reshape(-1)
    v = (p[:, 1:2] + (off // 3 - 1)).reshape(-1)
    d = p[:, 2:3].expand(-1, 9).reshape(-1)
    Rm = torch.as_tensor(np.asarray(cam.R, np.float64), device=DEV)
    t = torch.as_tensor(np.asarray(cam.t, np.float64), device=DEV)
    f = float(np.float32(cam.fx))
    xc = torch.stack([(u - cam.cx) / f, (v - cam.cy) / f, torch.ones_like(u)]) / d
    return u.long(), v.long(), d, Rm.T @ (xc - t[:, None]), f


def _nearest64(X, mean, k):
    best = torch.full((X.shape[1], 0), 0.0, dtype=torch.float64, device=DEV)
    idx = torch.zeros((X.shape[1], 0), dtype=torch.long, device=DEV)
    for a in range(0, mean.shape[1], 65536):
        m = mean[:, a:a + 65536]
        d2 = sum((X[i][:, None] - m[i][None]) ** 2 for i in range(3))
        best = torch.cat([best, d2], 1)
        idx = torch.cat([idx, torch.arange(a, a + m.shape[1], device=DEV)
                         .expand(X.shape[1], -1)], 1)
        best, o = torch.topk(best, min(k, best.shape[1]), 1, largest=False)
        idx = idx.gather(1, o)
    return best, idx


def _exact_insert(case, seed):
    s = prepare(case, seed)
    s.seed = seed
    n = case["n"]
    u, v, d, X, f = _candidates64(s, case)
    mean = s.params.data[0:3, :n].double()
    data = s.params.data.double()
    col = s.img[:, v, u].double()
    out = {}
    if case["kind"] == "distance":
        d2, _ = _nearest64(X, mean, 1)
        keep = d2[:, 0] > float(np.float32(0.02)) ** 2
        init = torch.cat([torch.log(1.0 / (d * f)).expand(3, -1),
                          torch.zeros_like(d)[None], col], 0)
        out.update(nearest2=None, n_ins=None)
    else:
        d2, idx = _nearest64(X, mean, 8)
        dist = d2.sqrt().clamp_min(1e-6)
        wgt = 1.0 / dist
        rgb = s.params.data[11:14].double()
        fe = torch.empty(u.numel(), 32, dtype=torch.float64, device=DEV)
        pad = torch.nn.functional.pad(s.img.double(), (1, 1, 1, 1))
        for q in range(9):
            fe[:, 3 * q:3 * q + 3] = pad[:, v + q // 3, u + q % 3].T
        fe[:, 27] = d
        fe[:, 28] = dist.log().mean(1)
        for ch in range(3):
            fe[:, 29 + ch] = (wgt * rgb[ch][idx]).sum(1) / wgt.sum(1)
        net = s.mlp
        h = (fe - net.x_mu.double()) / net.x_sd.double()
        h = _mlp64(net.w.double(), h)
        init = (h * net.t_sd.double() + net.t_mu.double())
        keep = 1.0 - s.T[v, u].double() <= float(np.float32(0.9))
        out.update(feats=fe, idx=None, init=init, n_ins=None)
        init = init.T
    new = torch.cat([X, init[0:3], torch.tensor([1.0, 0, 0, 0], device=DEV,
                     dtype=torch.float64)[:, None].expand(4, X.shape[1]),
                     init[3:7]], 0)[:, keep]
    data[:, n:n + new.shape[1]] = new
    out["data"] = data
    return out


def _mlp64(w, x):
    at, h = 0, x
    for i, (a, b) in enumerate(((32, 64), (64, 64), (64, 7))):
        h = h @ w[at:at + a * b].reshape(a, b) + w[at + a * b:at + a * b + b]
        at += a * b + b
        if i < 2:
            h = torch.nn.functional.gelu(h)
    return h


def _exact_mlp(case, seed):
    s = prepare(case, seed)
    w = s.net.w.double().requires_grad_(True)
    loss = ((_mlp64(w, s.x.double()) - s.t.double()) ** 2).mean()
    g = torch.autograd.grad(loss, w)[0]
    m = 0.9 * s.net.m.double() + 0.1 * g
    v = 0.999 * s.net.v.double() + 0.001 * g * g
    k = s.net.step + 1
    new = w.detach() - 1e-3 * (m / (1 - 0.9 ** k)) / (
        (v / (1 - 0.999 ** k)).sqrt() + 1e-8)
    return {"w": new, "g": g, "m": m, "loss": loss.detach().reshape(1)}


def exact(case, seed):
    kind = case["kind"]
    if kind == "colour":
        return _exact_colour(case, seed)
    if kind in ("distance", "learned"):
        return _exact_insert(case, seed)
    if kind == "mlp":
        return _exact_mlp(case, seed)
    if case.get("views", 1) * case["width"] * case["height"] > 4_000_000:
        return None   # over 20 seconds
    if kind == "densify":
        rgb, T, _, _ = _exact_render(case, seed, False)
        return {"rgb": rgb, "T": T, "dom": None, "data": None, "n_split": None}
    rgb, T, grad, loss = _exact_render(case, seed, True)
    if kind == "window":
        # Planar regulariser: mean of max(floor, smallest scale).
        ls = _scene(case, seed)[1][3:6].double()
        lm, ax = ls.min(0)
        sm, n = lm.exp(), ls.shape[1]
        floor = float(np.float32(0.01))
        loss += float(sm.clamp_min(floor).mean())
        add = torch.where(sm > floor, sm / n, torch.zeros_like(sm))
        grad[3 + ax, torch.arange(n, device=DEV)] += add
    return {"rgb": rgb, "T": T, "nlast": None, "grad": grad,
            "loss": torch.tensor([loss], dtype=torch.float64)}
