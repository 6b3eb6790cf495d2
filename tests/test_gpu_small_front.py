"""The lists of a step of up to 4096 (view, Gaussian) ids come from one
work-group, those of larger ones from the scans and the radix sort.  The same
visible Gaussians through both, bit for bit: a scene as it is, and with enough
Gaussians behind the cameras appended for the general path (and some put in
front, so that every place moves).  Counts around multiples of 64 and 1024 and
the largest that fit; equal depths, which keep index order; nothing visible."""
import numpy as np
import pytest
import torch

import scenes
from parity import gpu_params, upstream_tensors

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2511_16144_amd as P
    c = P.Context(0)
    yield c
    c.close()


def run(ctx, prm, cams, ups, tile, order):
    import paper_2511_16144_amd as P
    outs, state = ctx.forward(prm, cams, P.Settings(tile=tile, order=order), want_n=True)
    g = ctx.backward(state, prm, ups)
    torch.cuda.synchronize()
    c = state.counts()
    state.release()
    return outs, g, {k: c[k] for k in ("n_visible", "n_pairs", "n_slots")}


@pytest.mark.parametrize("n,views,tile,order", [(1, 1, 16, 0), (2, 3, 16, 0), (63, 1, 16, 0), (64, 2, 32, 2),
                                                (65, 1, 8, 0), (512, 8, 32, 2), (1023, 1, 16, 0), (1024, 3, 16, 0),
                                                (1025, 1, 16, 0), (2047, 2, 16, 0), (4095, 1, 16, 0),
                                                (4096, 1, 32, 1)])
@pytest.mark.parametrize("kind", ["spread", "equal depths", "hidden"])
def test_both_paths(ctx, n, views, tile, order, kind):
    print(f"[case] n {n} views {views} tile {tile} {kind}", flush=True)
    wl = scenes.tiny_scene(40 + n, n, 97, 71, z_range=(1.0, 3.0), log_scale=(-3.5, 0.7))
    sc = wl.scene
    if kind == "equal depths":
        sc.means[:, 2] = np.float32(1.5) + np.float32(0.25) * (np.arange(n) % 3)
    if kind == "hidden":
        sc.means[:, 2] = -1.0
    cams = [wl.cams[0]] * views
    small = gpu_params(sc)
    ups = upstream_tensors(scenes.random_upstream(n, cams, feat_dim=16))
    front, back = 5, 4100   # more than 4096 ids with them
    cols = torch.arange(-front, n + back).clamp(0, n - 1).cuda()
    large = {k: v[..., cols].contiguous() for k, v in small.items()}
    hide = torch.ones(n + front + back, dtype=torch.bool, device="cuda")
    hide[front:front + n] = False
    large["means"][2, hide] = -2.0
    o1, g1, c1 = run(ctx, small, cams, ups, tile, order)
    o2, g2, c2 = run(ctx, large, cams, ups, tile, order)
    assert c1 == c2 and (kind != "hidden" or c1["n_visible"] == 0)
    if kind != "hidden" and n > 60:
        assert c1["n_visible"] > 0
    for a, b in zip(o1, o2):
        for k in a:
            assert torch.equal(a[k], b[k]), k
    for k in g1:
        if k == "twist":   # the blocks of 64 ids that its partial sums take lie the same (visible ids are compacted)
            assert torch.equal(g1[k], g2[k]), k
        else:
            assert torch.equal(g1[k], g2[k][..., front:front + n]), k
            assert bool((g2[k][..., hide] == 0).all()), k
