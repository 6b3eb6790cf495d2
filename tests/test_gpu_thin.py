"""The geometric gradients of thin Gaussians (up to 24 pixels long, half a pixel
across and tilted), each alone on its pixels: what the sums over their pixels and
blocks add to the error.  Their gradients are what the short axis leaves of the
sums: along the image's axes, sums rounded to FP32 lose the square of the axes'
ratio.

As for small Gaussians: a red Gaussian alone renders its FP32 alpha, the FP64 oracle
gets the upstream times (rendered alpha / its own alpha), so both sides sum the same
products; positions are exact in FP32 (multiples of 1/64 pixel).

Tolerance 4e-7 of the norm, from an emulation of the products' roundings, the six
sums of a block and their sum over the blocks over such scenes: up to 1.4e-7 with the
sums in the Gaussian's own frame (0.7e-7 with exact sums), to which the FP32 contribution
of a view and the result add at most 1.2e-7; 6e-7 to 1.2e-5 along the image's axes,
the largest of a scene's groups never below 1.2e-6."""
import numpy as np
import pytest
import torch

import scenes
from oracle import raster_fp64 as R
from parity import ambiguous, gpu_params, grad_errors, grads_np, to_np

pytestmark = pytest.mark.gpu
TOL = 4e-7
COLS, ROWS, CELL, FOCAL, DEPTH = 6, 5, 160, 512.0, 2.0


@pytest.fixture(scope="module")
def ctx():
    import paper_2511_16144_amd as P
    c = P.Context(0)
    yield c
    c.close()


def workload(seed, dtype):
    r = np.random.Generator(np.random.PCG64(seed))
    n, W, H = COLS * ROWS, COLS * CELL, ROWS * CELL
    at = lambda k: CELL * k + CELL / 2 + np.floor(64 * r.uniform(-4, 4, n)) / 64  # noqa: E731
    x, y = at(np.arange(n) % COLS), at(np.arange(n) // COLS)
    cx, cy = (W - 1) / 2.0, (H - 1) / 2.0
    means = np.stack([(x - cx) * DEPTH / FOCAL, (y - cy) * DEPTH / FOCAL, np.full(n, DEPTH)], 1).astype(np.float32)
    px = np.stack([np.exp(r.uniform(np.log(4), np.log(22), n)), np.exp(r.uniform(np.log(0.05), np.log(0.5), n)),
                   np.full(n, 0.05)], 1)
    th = r.uniform(0, np.pi, n)
    q = np.stack([np.cos(th / 2), 0 * th, 0 * th, np.sin(th / 2)], 1).astype(np.float32)
    rgb = np.zeros((n, 3), np.float32)
    rgb[:, 0] = 1.0
    sc = scenes.Scene(means, np.log(px * DEPTH / FOCAL).astype(np.float32), q, r.normal(0.5, 0.5, n).astype(np.float32),
                      rgb, np.zeros((n, 16), np.float32), dtype)
    return sc, [scenes.Camera(W, H, FOCAL, FOCAL, cx, cy, np.eye(3, dtype=np.float32), np.zeros(3, np.float32))]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("mode", ["given", "L1"])
def test_thin(ctx, mode, dtype):
    import paper_2511_16144_amd as P
    for seed in (1, 2):
        sc, cams = workload(seed, dtype)
        W, H = cams[0].width, cams[0].height
        ref = R.render(sc, cams, R.Settings())[0]
        amb = ambiguous({**ref["margin"], "z": np.full((H, W), np.inf)})   # (no two share a pixel)
        prm = gpu_params(sc)
        outs, state = ctx.forward(prm, cams, P.Settings(), want_n=True)
        out = to_np(outs)[0]
        assert out["n"].max() == 1 and np.array_equal(out["n"][~amb], ref["n"][~amb])
        r = np.random.Generator(np.random.PCG64(seed + 50))
        g = r.normal(size=(H, W)).astype(np.float32)
        if mode == "given":
            g[amb] = 0.0
            up = [{k: torch.zeros_like(outs[0][k]) for k in ("rgb", "depth", "feat")}]
            up[0]["rgb"][0] = torch.as_tensor(g)
            got = ctx.backward(state, prm, up)
        else:   # weight 3 H W: the upstream is the residual's sign
            g = np.where(amb, 0.0, np.sign(g)).astype(np.float32)
            tg = [{k: outs[0][k].clone() for k in ("rgb", "depth", "feat")}]
            tg[0]["rgb"][0] -= torch.as_tensor(g).cuda()
            got = ctx.backward_l1(state, prm, outs, tg, (3.0 * H * W, 0.0, 0.0))
        got = grads_np(got)
        state.release()
        a64, a32 = ref["rgb"][0], out["rgb"][0].astype(np.float64)
        u = np.zeros((20, H, W))
        u[0] = np.where(a64 > 0, g * a32 / np.where(a64 > 0, a64, 1.0), 0.0)
        err = grad_errors(got, R.vjp(sc, cams, [u], R.Settings()), np.zeros(sc.n, bool))
        print(f"  {mode} {dtype} seed {seed}:", {k: "%.2e" % err[k][0] for k in err}, flush=True)
        for k in ("means", "log_scales", "quats", "logits"):
            assert err[k][0] <= TOL, (seed, k, err[k])
