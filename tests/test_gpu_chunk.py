"""settings.chunk = 8, which is accepted, against chunk = 4: a step in every form
of the backward (given upstream, fused L1, captured with D-SSIM), bit for bit."""
import numpy as np
import pytest
import torch

import scenes
from gpu_helpers import GraphRun
from parity import gpu_params, grads_np, to_np, upstream_tensors

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2511_16144_amd as P
    c = P.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_chunk_8_equals_chunk_4(ctx, dtype):
    import paper_2511_16144_amd as P
    wl = scenes.tiny_scene(3, 150, 77, 61)
    if dtype == "bf16":
        wl.scene.rgb, wl.scene.feat, wl.scene.dtype = (scenes.round_bf16(wl.scene.rgb),
                                                       scenes.round_bf16(wl.scene.feat), "bf16")
    prm, res = gpu_params(wl.scene), []
    tg = [{k: torch.as_tensor(getattr(t, k)).cuda() for k in ("rgb", "depth", "feat")} for t in wl.targets]
    for chunk in (4, 8):
        st = P.Settings(chunk=chunk)
        outs, state = ctx.forward(prm, wl.cams, st, want_n=True)
        g = [grads_np(ctx.backward(state, prm, upstream_tensors(scenes.random_upstream(1, wl.cams)))),
             grads_np(ctx.backward_l1(state, prm, outs, tg, (1.0, 1.0, 1.0)))]
        state.release()
        run = GraphRun(ctx, wl, st, ssim_lambda=0.2)
        assert run.rc == 0, P.lib().lgs_last_error(ctx._h).decode()
        run.launch()
        assert run.status() == 0
        res.append(to_np(outs) + g + [run.snapshot()[1]])
        run.destroy()
    for a, b in zip(*res):
        for k in a:
            assert np.array_equal(a[k], b[k]), k
