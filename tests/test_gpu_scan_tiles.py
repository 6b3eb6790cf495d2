"""The offset scans take whole blocks of 2048 ids 16 bytes at a time and the
last, part-filled one id by id.  Visible counts around one and two blocks, in
calls of more than 4096 ids (which take the scans), against calls of just the
visible Gaussians (one work-group does their lists), bit for bit."""
import pytest
import torch

import scenes
from parity import gpu_params, upstream_tensors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1, 2047, 2048, 2049, 4095, 4096])
def test_block_edges(m):
    import paper_2511_16144_amd as P
    print(f"[case] {m} visible", flush=True)
    ctx = P.Context(0)
    wl = scenes.tiny_scene(300, 4096, 97, 71, z_range=(1.0, 3.0), log_scale=(-3.5, 0.3))
    wl.scene.means[:, :2] *= 0.3   # every Gaussian in view
    full = gpu_params(wl.scene)
    full["logits"].clamp_(min=-1.0)
    small = {k: v[..., :m].contiguous() for k, v in full.items()}
    large = {k: torch.cat([v[..., :m], v[..., :1].expand(*v.shape[:-1], 4200)], -1).contiguous()
             for k, v in full.items()}
    large["means"][2, m:] = -2.0
    ups = upstream_tensors(scenes.random_upstream(1, wl.cams[:1], feat_dim=16))
    got = []
    for p in (small, large):
        outs, state = ctx.forward(p, wl.cams[:1], P.Settings(), want_n=True)
        g = ctx.backward(state, p, ups)
        torch.cuda.synchronize()
        assert state.counts()["n_visible"] == m
        state.release()
        got.append((outs[0], g))
    for k in got[0][0]:
        assert torch.equal(got[0][0][k], got[1][0][k]), k
    for k, a in got[0][1].items():
        b = got[1][1][k]
        assert torch.equal(a, b if k == "twist" else b[..., :m]), k
    ctx.close()
