"""The geometric gradients of Gaussians of about a pixel and less, each alone on
its pixels: what the backward adds to the error by summing over the pixels.

A red Gaussian alone on its pixels renders its FP32 alpha, and its gradients
are sums of upstream x alpha times moments of the pixel's offset.  The FP64
oracle gets the upstream times (rendered alpha / its own alpha), so that both
sides sum the same products; positions are exact in FP32 (multiples of 1/64
pixel).  What is left is the rounding of T / (1 - alpha) and of each product (3
roundings of 2^-24), of the sums, of the six results and of the parameters'.

Tolerance 2e-7 of the norm, from an emulation of these steps over the scenes
below: 0.8e-7 to 1.1e-7 with exact sums, at most 1.3e-7 with products in FP32
about the mean and a tree of additions; FP32 sums about centres apart from the
mean that are then moved to it lose up to 5.8e-7 (log_scales, quats)."""
import numpy as np
import pytest
import torch

import scenes
from oracle import raster_fp64 as R
from parity import ambiguous, gpu_params, grad_errors, grads_np, to_np

pytestmark = pytest.mark.gpu
TOL = 2e-7
COLS, ROWS, CELL, FOCAL, DEPTH = 20, 15, 12, 128.0, 2.0


@pytest.fixture(scope="module")
def ctx():
    import paper_2511_16144_amd as P
    c = P.Context(0)
    yield c
    c.close()


def workload(seed, lo, hi, dtype):
    """One Gaussian of lo .. hi pixels in each cell of a grid, at least 8 pixels apart."""
    r = np.random.Generator(np.random.PCG64(seed))
    n, W, H = COLS * ROWS, COLS * CELL, ROWS * CELL
    at = lambda k: CELL * k + np.floor(64 * r.uniform(4, 8, n)) / 64  # noqa: E731
    x, y = at(np.arange(n) % COLS), at(np.arange(n) // COLS)
    cx, cy = (W - 1) / 2.0, (H - 1) / 2.0
    means = np.stack([(x - cx) * DEPTH / FOCAL, (y - cy) * DEPTH / FOCAL, np.full(n, DEPTH)], 1).astype(np.float32)
    scales = np.exp(r.uniform(np.log(lo), np.log(hi), (n, 3))) * DEPTH / FOCAL
    q = r.normal(size=(n, 4))
    rgb = np.zeros((n, 3), np.float32)
    rgb[:, 0] = 1.0
    sc = scenes.Scene(means, np.log(scales).astype(np.float32), (q / np.linalg.norm(q, axis=1, keepdims=True)).astype(
        np.float32), r.normal(0.5, 0.5, n).astype(np.float32), rgb, np.zeros((n, 16), np.float32), dtype)
    return sc, [scenes.Camera(W, H, FOCAL, FOCAL, cx, cy, np.eye(3, dtype=np.float32), np.zeros(3, np.float32))]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("lo,hi", [(0.2, 0.6), (0.5, 1.2)])
@pytest.mark.parametrize("mode", ["given", "L1"])
def test_moments(ctx, mode, lo, hi, dtype):
    import paper_2511_16144_amd as P
    for seed in (1, 2):
        sc, cams = workload(seed, lo, hi, dtype)
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
        print(f"  {mode} {lo}..{hi} px {dtype} seed {seed}:", {k: "%.2e" % err[k][0] for k in err}, flush=True)
        for k in ("means", "log_scales", "quats", "logits"):
            assert err[k][0] <= TOL, (seed, k, err[k])
