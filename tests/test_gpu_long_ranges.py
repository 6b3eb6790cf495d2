"""The per-Gaussian reduction gives a Gaussian with more than 512 block slots
to a whole work-group, whose four waves take windows of 64 slots in turn.
Gaussians that cover the whole frame, on frames of 255 to 1025 blocks (512 the
last that one half-wave sums, 576 a whole number of windows), next to small
ones, against the FP64 oracle; a second backward over the same state gives the
same bits (the first cleared the slots' marks)."""
import numpy as np
import pytest
import torch

import scenes
from oracle import raster_fp64 as R
from parity import TOL_F32, ambiguous, fmt, gpu_params, grad_errors, grads_np, mask_upstream, upstream_tensors

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2511_16144_amd as P
    c = P.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("w,h", [(8 * 17, 8 * 15), (8 * 32, 8 * 16), (8 * 171, 8 * 3), (8 * 24, 8 * 24),
                                 (8 * 41 - 3, 8 * 25 - 7)])
def test_covering_gaussians(ctx, w, h):
    import paper_2511_16144_amd as P
    print(f"[case] {w} x {h}", flush=True)
    n = 9
    wl = scenes.tiny_scene(700 + w + h, n, w, h, z_range=(1.0, 1.6), log_scale=(-3.5, 0.3))
    sc = wl.scene
    sc.logits = np.linspace(-3.0, -1.5, n).astype(np.float32)
    big = [1, 4, 8]
    sc.log_scales[big] = np.float32([[2.0, 2.1, 2.2], [2.5, 2.2, 2.0], [2.1, 2.1, 2.1]])
    ref = R.render(sc, wl.cams, R.Settings())
    amb = ambiguous(ref[0]["margin"])
    prm = gpu_params(sc)
    outs, state = ctx.forward(prm, wl.cams, P.Settings())
    blocks = ((w + 7) // 8) * ((h + 7) // 8)
    assert state.counts()["n_slots"] >= len(big) * blocks
    ups = mask_upstream(scenes.random_upstream(n, wl.cams, feat_dim=16), [amb])
    dev = upstream_tensors(ups)
    first = grads_np(ctx.backward(state, prm, dev))
    again = grads_np(ctx.backward(state, prm, dev))
    torch.cuda.synchronize()
    state.release()
    assert all(np.array_equal(first[k], again[k]) for k in first)
    err = grad_errors(first, R.vjp(sc, wl.cams, ups, R.Settings()), np.zeros(n, bool))
    print(f"  {blocks} blocks: " + fmt(err), flush=True)
    for k, (l2, mx) in err.items():
        assert l2 <= TOL_F32 and mx <= TOL_F32, (k, l2, mx)
