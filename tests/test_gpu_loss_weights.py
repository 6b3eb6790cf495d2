"""Weights of the mapping loss of either sign and zero, which the calls accept: the
fused L1 backward (eager and captured) and the captured D-SSIM step against the
backward of the upstream that the same weights give (lgs_loss, then
lgs_backward).

Tolerance 1e-5, as between those forms elsewhere: they form the depth and
feature gradients in different products."""
import numpy as np
import pytest
import torch

import scenes
from gpu_helpers import GraphRun
from parity import gpu_params, grads_np, rel_err

pytestmark = pytest.mark.gpu
WEIGHTS = [(1.0, 0.5, 2.0), (-1.0, -0.5, -2.0), (1.0, -0.5, 2.0), (1.0, 0.5, -2.0), (-1.0, 0.5, 0.0), (0.0, 0.0, -1.0)]


@pytest.fixture(scope="module")
def ctx():
    import paper_2511_16144_amd as P
    c = P.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_signs(ctx, dtype):
    import paper_2511_16144_amd as P
    wl = scenes.tiny_scene(11, 120, 61, 47)
    if dtype == "bf16":
        wl.scene.rgb, wl.scene.feat, wl.scene.dtype = (scenes.round_bf16(wl.scene.rgb),
                                                       scenes.round_bf16(wl.scene.feat), "bf16")
    prm, st = gpu_params(wl.scene), P.Settings()
    outs, state = ctx.forward(prm, wl.cams, st)
    # a quarter off the rendered images, so that every residual's sign is clear
    r = np.random.Generator(np.random.PCG64(4))
    tg = [{k: o[k] + torch.as_tensor(0.25 * r.choice([-1.0, 1.0], o[k].shape).astype(np.float32)).cuda()
           for k in ("rgb", "depth", "feat")} for o in outs]
    wl.targets = [scenes.Targets(*(t[k].cpu().numpy() for k in ("rgb", "depth", "feat"))) for t in tg]
    for w in WEIGHTS:
        fused = grads_np(ctx.backward_l1(state, prm, outs, tg, w))
        for lam in (0.0, 0.2):
            up, _ = ctx.loss(wl.cams, outs, tg, w, lam)
            ref = grads_np(ctx.backward(state, prm, up))
            wl.loss_w = w
            run = GraphRun(ctx, wl, st, ssim_lambda=lam)
            assert run.rc == 0, P.lib().lgs_last_error(ctx._h).decode()
            run.launch()
            assert run.status() == 0
            got = run.snapshot()[1]
            run.destroy()
            for k in ref:
                for g in [got] + ([fused] if lam == 0.0 else []):
                    l2, mx = rel_err(g[k], ref[k])
                    assert l2 <= 1e-5 and mx <= 1e-5, (w, lam, k, l2, mx)
    state.release()
