"""The mapping loss without its D-SSIM term over both orders of its work-groups
(mixed; depth and features first, where they fill the chip), against the FP64
oracle and bit for bit against one view at a time."""
import numpy as np
import pytest

import scenes
from oracle import loss_fp64 as LF
from test_gpu_loss import check_loss, gpu_loss

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2511_16144_amd as P
    c = P.Context(0)
    yield c
    c.close()


def images(seed, sizes, D):
    outs, tgts = scenes.loss_images(seed, sizes)
    k = -(-D // 16)
    outs = [{**o, "feat": np.concatenate([o["feat"]] * k)[:D].copy()} for o in outs]
    tgts = [scenes.Targets(t.rgb, t.depth, np.concatenate([t.feat[::-1]] * k)[:D].copy()) for t in tgts]
    return outs, tgts


@pytest.mark.parametrize("sizes", [[(640, 818)], [(641, 817), (33, 5)], [(640, 817)], [(64, 48), (1030, 510)]])
@pytest.mark.parametrize("D", [8, 16, 32])
def test_orders(ctx, sizes, D):
    # (a streaming work-group takes 2048 pixels: 256 of them from 640 x 818 on)
    outs, tgts = images(len(sizes) + D, sizes, D)
    g, terms = gpu_loss(ctx, sizes, outs, tgts, (1.0, 0.5, 2.0), 0.0)
    _, ref_terms, ref = LF.loss_and_upstream(outs, tgts, (1.0, 0.5, 2.0), 0.0)
    check_loss(g, terms, ref_terms, ref, f"D={D}")
    for v in range(len(sizes)):
        g1, t1 = gpu_loss(ctx, sizes[v:v + 1], outs[v:v + 1], tgts[v:v + 1], (1.0, 0.5, 2.0), 0.0)
        assert np.array_equal(g1[0], g[v]) and np.array_equal(t1[0], terms[v])
