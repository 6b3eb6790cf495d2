"""Timed cases of the rasterizer library: what a mapping program has it do.

Each case is one call (or one forward + backward pair) through the public
entry points of ``paper_2511_16144_amd``: mapping steps (eager and as a
captured graph, with and without D-SSIM), the autograd render, forward-only
renders, the mapping loss alone, the feature decoder and the pruning pass.
Scenes are seeded stand-ins for indoor RGB-D maps: Gaussians on the faces of
a 6 x 6 x 3 m room (or in a camera frustum, for the smallest maps) with 5 cm
scales.

``exact`` renders the same inputs in FP64 by the definition (per pixel, in
depth order) with torch alone.
"""
import ctypes as C
import math

import torch

import paper_2511_16144_amd as P
from paper_2511_16144_amd import binding as B

DEV = "cuda:0"
CUTOFF2 = 9.0
# constants of the settings as the FP32 values that the library receives
EPS2D, FOV, AMAX, AMIN, ZN, TEPS = (float(torch.tensor(x, dtype=torch.float32))
                                    for x in (0.3, 1.3, 0.99, 1.0 / 255.0, 0.2, 1e-4))
# An L1 residual has no gradient at 0, and next to 0 its sign is a matter of
# the last bit: targets are kept this far off the rendered values.
GAP = 1e-3


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def listed():
    base = {"scene": "room", "views": 1, "dtype": "f32", "D": 16, "tile": 16, "order": 0}
    tuned = {"tile": 32, "order": 2}
    return [
        # one mapping iteration on the first keyframes of a map: latency and launches
        {**base, "name": "step_tiny_f32", "kind": "step", "scene": "frustum", "n": 2000, "w": 128, "h": 96},
        # one mapping iteration over a single keyframe, default settings
        {**base, "name": "step_single_f32", "kind": "step", "n": 300_000, "w": 640, "h": 480},
        # the mapping iteration over a keyframe window, captured once and replayed
        {**base, **tuned, "name": "graph_window_bf16", "kind": "graph", "n": 500_000, "views": 8, "w": 640, "h": 480,
         "dtype": "bf16", "ssim": 0.0},
        # a large map and frame, photometric term with D-SSIM
        {**base, **tuned, "name": "graph_dssim_bf16", "kind": "graph", "n": 1_000_000, "w": 1200, "h": 680,
         "dtype": "bf16", "ssim": 0.2},
        # pose refinement and user-defined losses: torch autograd, any upstream, ragged frame
        {**base, "name": "autograd_ragged_f32", "kind": "autograd", "n": 60_000, "w": 333, "h": 251},
        {**base, "name": "autograd_bf16", "kind": "autograd", "n": 300_000, "w": 613, "h": 457, "dtype": "bf16"},
        # a viewer or a query: the largest map and frame, forward only
        {**base, **tuned, "name": "render_large_bf16", "kind": "render", "n": 2_000_000, "w": 1296, "h": 968,
         "dtype": "bf16"},
        # a wider language feature (four groups of 16 channels)
        {**base, "name": "step_feat64_bf16", "kind": "step", "n": 100_000, "w": 320, "h": 240, "dtype": "bf16",
         "D": 64},
        # the mapping loss with D-SSIM on the images of a keyframe window
        {"name": "loss_window", "kind": "loss", "views": 8, "w": 640, "h": 480, "D": 16, "ssim": 0.2},
        # feature distillation of a keyframe window through the decoder
        {"name": "decoder_window_bf16", "kind": "decoder", "views": 8, "w": 640, "h": 480, "C": 512,
         "dtype": "bf16"},
        # ... and of one small ragged frame with FP32 targets
        {"name": "decoder_small_f32", "kind": "decoder", "views": 1, "w": 157, "h": 119, "C": 256, "dtype": "f32"},
        # pruning of a whole map
        {"name": "prune_map_bf16", "kind": "prune", "n": 500_000, "dtype": "bf16", "k": 16},
    ]


def draw(rng):
    def log(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    kind = rng.choice(["step", "step", "graph", "graph", "autograd", "render", "loss", "decoder", "prune"])
    dtype = rng.choice(["f32", "bf16"])
    if kind == "prune":
        return {"kind": kind, "n": log(2000, 500_000), "dtype": dtype, "k": rng.choice([4, 8, 16, 16, 32])}
    w = log(96, 800)
    h = max(64, int(w * rng.uniform(0.5, 0.85)))
    views = rng.choice([1, 1, 2, 3, 6]) if w < 480 else rng.choice([1, 2])
    if kind == "decoder":
        return {"kind": kind, "views": views, "w": w, "h": h, "C": rng.choice([256, 512]), "dtype": dtype}
    if kind == "loss":
        return {"kind": kind, "views": views, "w": w, "h": h, "D": rng.choice([8, 16, 16, 32]),
                "ssim": rng.choice([0.0, 0.2, 0.2])}
    tile, order = rng.choice([(16, 0), (32, 2), (32, 2), (32, 1), (8, 0)])
    c = {"kind": kind, "scene": "room", "n": log(2000, 500_000), "views": views, "w": w, "h": h, "dtype": dtype,
         "D": rng.choice([8, 16, 16, 16, 32] if w * h * views < 150_000 else [16]), "tile": tile, "order": order}
    if kind == "graph":
        c["ssim"] = rng.choice([0.0, 0.0, 0.2])
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
class Camera:
    def __init__(self, w, h, f, R, t):
        self.width, self.height, self.fx, self.fy = w, h, f, f
        self.cx, self.cy = (w - 1) / 2.0, (h - 1) / 2.0
        self.R_cw, self.t_cw = R, t


def _f32(x):
    return float(torch.tensor(x, dtype=torch.float32))


def _yaw_camera(center, yaw, w, h, f):
    """A camera at `center` looking horizontally along yaw (z up)."""
    c, s = math.cos(yaw), math.sin(yaw)
    R = [[s, -c, 0.0], [0.0, 0.0, -1.0], [c, s, 0.0]]
    t = [-sum(R[i][j] * center[j] for j in range(3)) for i in range(3)]
    return Camera(w, h, _f32(f), [[_f32(x) for x in r] for r in R], [_f32(x) for x in t])


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _rand(g, *shape):
    return torch.rand(shape, generator=g, device=DEV)


def _randn(g, *shape):
    return torch.randn(shape, generator=g, device=DEV)


def _room_points(g, n):
    """Uniform on the six inner faces of [-3,3] x [-3,3] x [0,3], plus 2 cm of noise."""
    face = torch.bucketize(_rand(g, n), torch.tensor([0.25, 0.5, 0.625, 0.75, 0.875], device=DEV))
    a, b = _rand(g, n), _rand(g, n)
    u6, v6, v3 = 6 * a - 3, 6 * b - 3, 3 * b
    m3 = torch.full_like(a, 3.0)
    x = torch.stack([u6, u6, -m3, m3, u6, u6])
    y = torch.stack([v6, v6, u6, u6, -m3, m3])
    z = torch.stack([torch.zeros_like(a), m3, v3, v3, v3, v3])
    pick = lambda t: t.gather(0, face[None])[0]  # noqa: E731
    return torch.stack([pick(x), pick(y), pick(z)]) + 0.02 * _randn(g, 3, n)


def _cameras(case, seed):
    r = torch.Generator().manual_seed(int(seed) + 77)
    u = lambda: float(torch.rand((), generator=r))  # noqa: E731
    w, h, V = case["w"], case["h"], case["views"]
    if case["scene"] == "frustum":
        return [Camera(w, h, _f32(100.0 * w / 128), [[1.0, 0, 0], [0, 1.0, 0], [0, 0, 1.0]], [0.0, 0.0, 0.0])]
    if V == 1:
        return [_yaw_camera((4 * u() - 2, 4 * u() - 2, 1 + u()), 2 * math.pi * u(), w, h, 577.0 * w / 640)]
    cams, turn = [], 2 * math.pi * u()
    for v in range(V):   # a window on a circle, looking inward; every other keyframe at half the size
        a = turn + 2 * math.pi * v / V
        k = 1 if v % 2 == 0 else 2
        cams.append(_yaw_camera((2 * math.cos(a), 2 * math.sin(a), 1.5), a + math.pi, w // k, h // k,
                                577.0 * w / 640 / k))
    return cams


def _store(t, dtype):
    return t.to(torch.bfloat16) if dtype == "bf16" else t


def _gaussians(case, seed):
    g, n, D = _gen(seed), case["n"], case["D"]
    if case["scene"] == "frustum":
        z = (1 + 124 * _rand(g, n)) ** (1.0 / 3.0)
        f = 100.0 * case["w"] / 128
        means = torch.stack([(_rand(g, n) - 0.5) * case["w"] * z / f, (_rand(g, n) - 0.5) * case["h"] * z / f, z])
    else:
        means = _room_points(g, n)
    return {"means": means, "log_scales": -3.0 + 0.5 * _randn(g, 3, n),
            "quats": torch.nn.functional.normalize(_randn(g, 4, n), dim=0), "logits": _randn(g, n),
            "rgb": _store(_rand(g, 3, n), case["dtype"]),
            "feat": _store(torch.nn.functional.normalize(_randn(g, D, n), dim=0), case["dtype"])}


def _frames(case, seed, cams, far=6.0):
    """Observed images (or any images of those ranges) of every view."""
    g, out = _gen(seed), []
    for c in cams:
        hw = (c.height, c.width)
        out.append({"rgb": _rand(g, 3, *hw), "depth": 0.5 + (far - 0.5) * _rand(g, *hw),
                    "feat": torch.nn.functional.normalize(_randn(g, case["D"], *hw), dim=0)})
    return out


def _upstream(case, seed, cams):
    g = _gen(seed)
    return [{"rgb": _randn(g, 3, c.height, c.width), "depth": _randn(g, c.height, c.width),
             "feat": _randn(g, case["D"], c.height, c.width), "T": _randn(g, c.height, c.width)} for c in cams]


def _apart(t, y):
    """Targets t, moved off the rendered values y where they are closer than GAP."""
    d = t - y
    return torch.where(d.abs() < GAP, t + torch.where(d >= 0, GAP, -GAP), t)


def _loss_cameras(case):
    return [Camera(case["w"] // (1 + v % 2), case["h"] // (1 + v % 2), 1.0, [[1.0, 0, 0], [0, 1.0, 0], [0, 0, 1.0]],
                   [0.0, 0.0, 0.0]) for v in range(case["views"])]


def _loss_images(case, seed):
    cams = _loss_cameras(case)
    tgt = _frames(case, seed, cams)
    g = _gen(seed + 500)
    out = [{"rgb": (t["rgb"] + 0.1 * _randn(g, *t["rgb"].shape)).clamp(0, 1),
            "depth": t["depth"] + 0.3 * _randn(g, *t["depth"].shape),
            "feat": t["feat"] + 0.3 * _randn(g, *t["feat"].shape)} for t in tgt]
    return cams, out, tgt


def _decoder_inputs(case, seed):
    """Feature maps, decoder and extractor features; the residuals have a gap of 0.02 around 0 (see GAP)."""
    g, Cd = _gen(seed), case["C"]
    W, b = 0.25 * _randn(g, Cd, 16), 0.05 * _randn(g, Cd)
    feats, tgts = [], []
    for c in _loss_cameras(case):
        f = 0.25 * _randn(g, 16, c.height, c.width)
        r = 0.3 * _randn(g, Cd, c.height, c.width)
        r = r + torch.where(r >= 0, 0.02, -0.02)
        r += (W @ f.reshape(16, -1) + b[:, None]).reshape(Cd, c.height, c.width)
        feats.append(f)
        tgts.append(_store(r, case["dtype"]))
    return W, b, feats, tgts


def _prune_inputs(case, seed):
    """A room whose Gaussians carry the noisy feature of the object they belong to."""
    p = _gaussians({**case, "scene": "room", "D": 16}, seed)
    g, n = _gen(seed + 900), case["n"]
    centres = torch.tensor([6.0, 6.0, 3.0], device=DEV)[:, None] * _rand(g, 3, 64) - torch.tensor(
        [3.0, 3.0, 0.0], device=DEV)[:, None]
    best, obj = torch.full((n,), math.inf, device=DEV), torch.zeros(n, dtype=torch.long, device=DEV)
    for k in range(64):
        d = ((p["means"] - centres[:, k:k + 1]) ** 2).sum(0)
        obj = torch.where(d < best, k, obj)
        best = torch.minimum(best, d)
    f = torch.nn.functional.normalize(_randn(g, 16, 64), dim=0)[:, obj] + 0.08 * _randn(g, 16, n)
    p["feat"] = _store(torch.nn.functional.normalize(f, dim=0), case["dtype"])
    return p


# ---------------------------------------------------------------------------
# what a program keeps, and one pass
# ---------------------------------------------------------------------------
class Graph:
    """A captured mapping step bound to its image and gradient buffers."""

    def __init__(self, ctx, settings, params, cams, targets, ssim):
        self.h, self.ctx, self.keep = None, ctx, (params, targets)
        dev, D = params["means"].device, params["feat"].shape[0]
        self.outs = [{"rgb": torch.empty((3, c.height, c.width), device=dev),
                      "depth": torch.empty((c.height, c.width), device=dev),
                      "feat": torch.empty((D, c.height, c.width), device=dev),
                      "T": torch.empty((c.height, c.width), device=dev)} for c in cams]
        V = len(cams)
        self.grads, gr = B._grad_buffers(params["logits"].shape[0], V, dev, D)
        shapes = [(c.height, c.width) for c in cams]
        g = B.gaussians_c(*(params[k] for k in ("means", "log_scales", "quats", "logits", "rgb", "feat")))
        st, h = settings.to_c(), C.c_void_p()
        rc = B.lib().lgs_graph_create(ctx._h, C.byref(st), C.byref(g), V, (B.lgs_camera * V)(*map(B.camera_c, cams)),
                                      B._images_c(targets, shapes, False), (C.c_float * 3)(1.0, 1.0, 1.0),
                                      C.c_float(ssim), B._images_c(self.outs, shapes, True), C.byref(gr), 0,
                                      B._stream(), C.byref(h))
        if rc != B.LGS_OK:
            raise B.LgsError(rc, B.lib().lgs_last_error(ctx._h).decode())
        self.h = h

    def launch(self):
        rc = B.lib().lgs_graph_launch(self.h, B._stream())
        if rc != B.LGS_OK:
            raise B.LgsError(rc, B.lib().lgs_last_error(self.ctx._h).decode())

    def __del__(self):
        if self.h:
            B.lib().lgs_graph_destroy(self.h)
            self.h = None


def prepare(case, seed):
    s = {"case": case, "ctx": P.Context(0)}
    kind = case["kind"]
    if kind == "loss":
        s["cams"], s["outs"], s["targets"] = _loss_images(case, seed)
    elif kind == "decoder":
        s["W"], s["b"], s["feats"], s["targets"] = _decoder_inputs(case, seed)
    elif kind == "prune":
        s["params"] = _prune_inputs(case, seed)
    else:
        s["params"], s["cams"] = _gaussians(case, seed), _cameras(case, seed)
        s["settings"] = P.Settings(tile=case["tile"], order=case["order"])
        if kind in ("step", "graph"):
            outs, state = s["ctx"].forward(s["params"], s["cams"], s["settings"])
            state.release()
            s["targets"] = [{k: _apart(t[k], o[k]) for k in t}
                            for t, o in zip(_frames(case, seed + 300, s["cams"]), outs)]
        if kind == "graph":
            s["graph"] = Graph(s["ctx"], s["settings"], s["params"], s["cams"], s["targets"], case["ssim"])
        if kind == "autograd":
            s["up"] = _upstream(case, seed + 300, s["cams"])
            s["storage"] = s["params"]["rgb"].dtype   # FP32 masters, handed over in the storage type
            s["params"] = {k: t.float().requires_grad_(True) for k, t in s["params"].items()}
    return s


def run(s):
    kind, ctx = s["case"]["kind"], s["ctx"]
    if kind == "step":
        outs, state = ctx.forward(s["params"], s["cams"], s["settings"])
        grads = ctx.backward_l1(state, s["params"], outs, s["targets"], (1.0, 1.0, 1.0))
        state.release()
        return {"images": outs, "grads": grads}
    if kind == "graph":
        s["graph"].launch()
        return {"images": s["graph"].outs, "grads": s["graph"].grads}
    if kind == "render":
        outs, state = ctx.forward(s["params"], s["cams"], s["settings"])
        state.release()
        return {"images": outs}
    if kind == "autograd":
        p = s["params"]
        twist = torch.zeros((len(s["cams"]), 6), device=DEV, requires_grad=True)
        outs = P.render(ctx, p, s["cams"], s["settings"], twist=twist, storage=s["storage"])
        keys = ("rgb", "depth", "feat", "T")
        grads = torch.autograd.grad([o[k] for o in outs for k in keys], [*p.values(), twist],
                                    [u[k] for u in s["up"] for k in keys])
        return {"images": outs, "grads": dict(zip([*p, "twist"], grads))}
    if kind == "loss":
        grad, terms = ctx.loss(s["cams"], s["outs"], s["targets"], (1.0, 1.0, 1.0), s["case"]["ssim"])
        return {"grad": grad, "terms": terms}
    if kind == "decoder":
        if len(s["feats"]) == 1:
            loss, gf, gw, gb = ctx.decoder_l1(s["feats"][0], s["W"], s["b"], s["targets"][0])
            gf = [gf]
        else:
            loss, gf, gw, gb = ctx.decoder_l1_views(s["feats"], s["W"], s["b"], s["targets"])
        return {"loss": loss, "feat": gf, "weight": gw, "bias": gb}
    mask, counts = ctx.prune(s["params"], k=s["case"]["k"])
    return {"mask": mask, "counts": counts}


# ---------------------------------------------------------------------------
# the work of a pass
# ---------------------------------------------------------------------------
def work(case):
    """Inputs read once, outputs written once; FP32 operations of the per-pixel definition (FMA = 2): 60 per
    contributing (pixel, Gaussian) in the forward, 119 in the backward, 16 more per channel beyond 16 features.
    A pixel has about n pi (2.5 s)^2 / (room surface) contributors (s = 5 cm, 144 m^2), at most about 110 before
    its transmittance ends."""
    kind, e = case["kind"], 2 if case.get("dtype") == "bf16" else 4
    if kind == "prune":
        n = case["n"]
        near = n * 4.0 / 3.0 * math.pi * 0.02 ** 3 / (144.0 * 0.05)   # within tau_dist of a Gaussian
        return {"bytes": n * (3 * 4 + 4 + 12 + 16 * e + 1), "flops": n * (8 * near + 70 * min(near, case["k"]))}
    px = sum((case["w"] // (1 + v % 2)) * (case["h"] // (1 + v % 2)) for v in range(case["views"]))
    if kind == "decoder":
        Cd = case["C"]
        return {"bytes": px * (Cd * e + 128) + 2 * 4 * 17 * Cd, "flops": px * 3 * 2 * 16 * Cd}
    D = case["D"]
    if kind == "loss":
        return {"bytes": px * (4 + D) * 12, "flops": px * (3 * (390 if case["ssim"] else 3) + 3 * (1 + D))}
    n = case["n"]
    per = 15.0 if case["scene"] == "frustum" else min(110.0, n * 3.4e-4)
    image = 4 * (5 + D)
    by = n * (44 + (3 + D) * e) + px * image
    fl = px * per * (60 + 2 * (D - 16))
    if kind != "render":
        by += px * 4 * (4 + D) + n * 4 * (14 + D)
        fl += px * per * (119 + 4 * (D - 16))
    if case.get("ssim"):
        fl += px * 3 * 390
    return {"bytes": by, "flops": fl}


# ---------------------------------------------------------------------------
# the same in FP64
# ---------------------------------------------------------------------------
def _skew(a):
    o = torch.zeros((), dtype=torch.float64, device=DEV)
    return torch.stack([torch.stack([o, -a[2], a[1]]), torch.stack([a[2], o, -a[0]]), torch.stack([-a[1], a[0], o])])


def _project64(p, cam, xi):
    """Screen mean [2,n], covariance and conic [3,n], opacity and depth in FP64; xi: the left pose twist at 0."""
    R = torch.tensor(cam.R_cw, dtype=torch.float64, device=DEV)
    t = torch.tensor(cam.t_cw, dtype=torch.float64, device=DEV)
    K = _skew(xi[3:])
    R, t = R + K @ R, t + K @ t + xi[:3]
    q = p["quats"] / p["quats"].norm(dim=0, keepdim=True)
    w, x, y, z = q
    Rq = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                      2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                      2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)]).reshape(3, 3, -1)
    M = Rq * p["log_scales"].exp()[None]
    M = (R @ M.reshape(3, -1)).reshape(3, 3, -1)
    xc = R @ p["means"] + t[:, None]
    zc = xc[2]
    u, v = xc[0] / zc, xc[1] / zc
    fx, fy, cx, cy = float(cam.fx), float(cam.fy), _f32(cam.cx), _f32(cam.cy)
    lx = FOV * max(cx + 0.5, cam.width - 0.5 - cx) / fx
    ly = FOV * max(cy + 0.5, cam.height - 0.5 - cy) / fy
    m1 = (fx / zc) * M[0] - (fx * u.clamp(-lx, lx) / zc) * M[2]
    m2 = (fy / zc) * M[1] - (fy * v.clamp(-ly, ly) / zc) * M[2]
    a, b, c = (m1 * m1).sum(0) + EPS2D, (m1 * m2).sum(0), (m2 * m2).sum(0) + EPS2D
    det = a * c - b * b
    return (torch.stack([fx * u + cx, fy * v + cy]), torch.stack([a, c]), torch.stack([c / det, -b / det, a / det]),
            torch.sigmoid(p["logits"]), zc)


def _tile64(mu, con, o, app, px, py, step=768):
    """Colours [pixels, channels] and final transmittance of one pixel tile over its Gaussians in depth order."""
    Y = torch.zeros((px.numel(), app.shape[1]), dtype=torch.float64, device=DEV)
    T = torch.ones(px.numel(), dtype=torch.float64, device=DEV)
    end = T
    for k in range(0, o.numel(), step):
        s = slice(k, k + step)
        dx, dy = px[:, None] - mu[0, s], py[:, None] - mu[1, s]
        m2 = con[0, s] * dx * dx + 2 * con[1, s] * dx * dy + con[2, s] * dy * dy
        raw = o[s] * torch.exp(-0.5 * m2)
        alpha = torch.where(raw > AMAX, AMAX, raw)
        alpha = torch.where((m2 <= CUTOFF2) & (alpha >= AMIN), alpha, 0.0)
        after = T[:, None] * torch.exp(torch.cumsum(torch.log1p(-alpha), 1))
        before = torch.cat([T[:, None], after[:, :-1]], 1)
        keep = after >= TEPS
        Y = Y + torch.where(keep, alpha * before, 0.0) @ app[s]
        n_kept = keep.sum(1)
        last = after.gather(1, (n_kept - 1).clamp(min=0)[:, None])[:, 0]
        end = torch.where(n_kept > 0, last, end)
        T = after[:, -1]
        if not bool((T >= TEPS).any()):
            break
    return Y, end


def _render64(p, cam, xi, upstream=None, side=32):
    """One view; with `upstream(Y, T, rows, columns)` -> (dL/dY, dL/dT) also the gradient, accumulated in the
    leaves p and xi.  Returns the image [4 + D, H, W] and T [H, W]."""
    mu, cov, con, o, z = _project64(p, cam, xi)
    app = torch.cat([p["rgb"], z[None], p["feat"]]).T
    with torch.no_grad():
        r2 = torch.minimum(torch.full_like(o, CUTOFF2), 2 * torch.log(o / AMIN))
        vis = (z > ZN) & (o >= AMIN) & (r2 >= 0)
        r = torch.sqrt(r2.clamp(min=0) * cov) + 0.01
        lo, hi = mu - r, mu + r
        vis &= (hi[0] >= 0) & (hi[1] >= 0) & (lo[0] <= cam.width - 1) & (lo[1] <= cam.height - 1)
        idx = vis.nonzero()[:, 0]
        idx = idx[torch.sort(z[idx], stable=True)[1]]
        lo, hi = lo[:, idx], hi[:, idx]
        img = torch.empty((app.shape[1], cam.height, cam.width), dtype=torch.float64, device=DEV)
        Tim = torch.empty((cam.height, cam.width), dtype=torch.float64, device=DEV)
    leaves = [t.detach() for t in (mu, con, o, app)]
    sums = [torch.zeros_like(t) for t in leaves]
    for y0 in range(0, cam.height, side):
        y1 = min(y0 + side, cam.height)
        row = ((hi[1] >= y0) & (lo[1] <= y1 - 1)).nonzero()[:, 0]
        for x0 in range(0, cam.width, side):
            x1 = min(x0 + side, cam.width)
            at = idx[row[(hi[0][row] >= x0) & (lo[0][row] <= x1 - 1)]]
            py, px = torch.meshgrid(torch.arange(y0, y1, device=DEV, dtype=torch.float64),
                                    torch.arange(x0, x1, device=DEV, dtype=torch.float64), indexing="ij")
            part = [leaves[0][:, at], leaves[1][:, at], leaves[2][at], leaves[3][at]]
            if upstream is not None:
                part = [t.requires_grad_(True) for t in part]
            with torch.set_grad_enabled(upstream is not None):
                Y, T = _tile64(*part, px.reshape(-1), py.reshape(-1))
                if upstream is not None and at.numel():
                    gY, gT = upstream(Y.detach(), T.detach(), slice(y0, y1), slice(x0, x1))
                    got = torch.autograd.grad((Y * gY).sum() + (T * gT).sum(), part)
            img[:, y0:y1, x0:x1] = Y.detach().T.reshape(-1, y1 - y0, x1 - x0)
            Tim[y0:y1, x0:x1] = T.detach().reshape(y1 - y0, x1 - x0)
            if upstream is not None and at.numel():
                for k, gk in enumerate(got):
                    sums[k].index_add_(1 if k < 2 else 0, at, gk)
    if upstream is not None:
        # (a view's invisible Gaussians have no part in it; their infinities stay out)
        seen = [t[:, idx] if k < 2 else t[idx] for k, t in enumerate((mu, con, o, app))]
        torch.autograd.backward(seen, [t[:, idx] if k < 2 else t[idx] for k, t in enumerate(sums)])
    return img, Tim


def _blur64(x):
    """11 x 11 Gaussian window (sigma 1.5), zeros outside the image."""
    w = [math.exp(-(k * k) / 4.5) for k in range(-5, 6)]
    w = [k / sum(w) for k in w]
    for d in (1, 2):
        pad = torch.nn.functional.pad(x, (5, 5, 0, 0) if d == 2 else (0, 0, 5, 5))
        x = sum(wk * pad.narrow(d, k, x.shape[d]) for k, wk in enumerate(w))
    return x


def _terms64(o, t, ssim):
    """The loss terms (mean |I - I*|, 1 - SSIM, mean |D - D*|, mean |F - F*|) of one view."""
    x, y = o["rgb"], t["rgb"]
    term = torch.zeros((), dtype=torch.float64, device=DEV)
    if ssim:
        mx, my = _blur64(x), _blur64(y)
        vx, vy, cxy = _blur64(x * x) - mx * mx, _blur64(y * y) - my * my, _blur64(x * y) - mx * my
        term = 1 - (((2 * mx * my + 1e-4) * (2 * cxy + 9e-4)) / ((mx * mx + my * my + 1e-4) * (vx + vy + 9e-4))).mean()
    return [(x - y).abs().mean(), term, (o["depth"] - t["depth"]).abs().mean(), (o["feat"] - t["feat"]).abs().mean()]


def _loss64(o, t, ssim):
    lam = _f32(ssim)
    a, b, c, d = _terms64(o, t, ssim)
    return (1 - lam) * a + lam * b + c + d


def _loss_grad64(img, t, ssim):
    o = {"rgb": img[:3].clone().requires_grad_(True), "depth": img[3].clone().requires_grad_(True),
         "feat": img[4:].clone().requires_grad_(True)}
    t = {k: _apart(t[k].double(), o[k].detach()) for k in t}
    g = torch.autograd.grad(_loss64(o, t, ssim), list(o.values()))
    return torch.cat([g[0], g[1][None], g[2]])


def _exact_render(case, seed):
    cams = _cameras(case, seed)
    p = {k: t.double().requires_grad_(True) for k, t in _gaussians(case, seed).items()}
    kind, images, twists = case["kind"], [], []
    frames = _frames(case, seed + 300, cams) if kind in ("step", "graph") else None
    ups = _upstream(case, seed + 300, cams) if kind == "autograd" else None
    for v, cam in enumerate(cams):
        xi = torch.zeros(6, dtype=torch.float64, device=DEV, requires_grad=True)
        if kind == "render":
            with torch.no_grad():
                img, T = _render64(p, cam, xi)
        else:
            if kind == "autograd":
                u = torch.cat([ups[v]["rgb"], ups[v]["depth"][None], ups[v]["feat"]]).double()
                uT = ups[v]["T"].double()
            else:
                with torch.no_grad():
                    img, T = _render64(p, cam, xi)
                u, uT = _loss_grad64(img, frames[v], case.get("ssim", 0.0)), torch.zeros_like(T)
            img, T = _render64(p, cam, xi, lambda Y, Tt, r, c: (u[:, r, c].reshape(u.shape[0], -1).T,
                                                                uT[r, c].reshape(-1)))
            twists.append(xi.grad)
        images.append({"rgb": img[:3], "depth": img[3], "feat": img[4:], "T": T})
    if kind == "render":
        return {"images": images}
    return {"images": images, "grads": {**{k: t.grad for k, t in p.items()}, "twist": torch.stack(twists)}}


def exact(case, seed):
    kind = case["kind"]
    if kind == "prune":   # a mask and counts: whole numbers
        return None
    if kind == "loss":
        _, outs, tgts = _loss_images(case, seed)
        grads, terms = [], []
        for o, t in zip(outs, tgts):
            o = {k: x.double().requires_grad_(True) for k, x in o.items()}
            t = {k: x.double() for k, x in t.items()}
            grads.append(dict(zip(o, torch.autograd.grad(_loss64(o, t, case["ssim"]), list(o.values())))))
            terms.append(torch.stack([x.detach() for x in _terms64(o, t, case["ssim"])]))
        return {"grad": grads, "terms": torch.stack(terms)}
    if kind == "decoder":
        W, b, feats, tgts = _decoder_inputs(case, seed)
        W, b = W.double(), b.double()
        loss, gw, gb, gfs = 0.0, torch.zeros_like(W), torch.zeros_like(b), []
        for f, t in zip(feats, tgts):
            n, f2, t2 = f[0].numel(), f.reshape(16, -1).double(), t.reshape(case["C"], -1)
            gf = torch.empty_like(f2)
            for k in range(0, n, 1 << 16):
                s = slice(k, k + (1 << 16))
                d = W @ f2[:, s] + b[:, None] - t2[:, s].double()
                loss = loss + d.abs().sum() / (case["C"] * n)
                r = d.sign() / (case["C"] * n)
                gf[:, s] = W.T @ r
                gw += r @ f2[:, s].T
                gb += r.sum(1)
            gfs.append(gf.reshape(f.shape))
        return {"loss": loss.reshape(1), "feat": gfs, "weight": gw, "bias": gb}
    return _exact_render(case, seed)
