"""The D-SSIM gradient's rounding where it is largest: smooth images, whose window
variances are small against the squares they are differences of.

Tolerance 1.1e-5 of the norm, from an emulation of the kernel's FP32 steps on
these images: 0.78e-5 with the variances' sum taken as twice the covariance plus
the variance of the difference; 1.4e-5 with separate sums of X^2 and Y^2, 1.6e-5
with one of X^2 + Y^2."""
import numpy as np
import pytest

import scenes
from oracle import loss_fp64 as LF
from parity import rel_err
from test_gpu_loss import gpu_loss

pytestmark = pytest.mark.gpu
TOL = 1.1e-5


@pytest.fixture(scope="module")
def ctx():
    import paper_2511_16144_amd as P
    c = P.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("W,H", [(96, 96), (157, 119)])
def test_smooth_images(ctx, W, H):
    r = np.random.Generator(np.random.PCG64(W))
    y, x = np.mgrid[0:H, 0:W] / 96.0
    base = np.stack([0.5 + 0.3 * np.sin(5 * x + c) * np.cos(4 * y) for c in range(3)])
    flat = {"depth": np.ones((H, W), np.float32), "feat": np.ones((16, H, W), np.float32)}
    out = {"rgb": (base + 0.02 * r.normal(size=base.shape)).astype(np.float32), **flat}
    tgt = scenes.Targets(base.astype(np.float32), flat["depth"], flat["feat"])
    # lambda 1: the colour gradient is the D-SSIM term's alone
    g, terms = gpu_loss(ctx, [(W, H)], [out], [tgt], (1.0, 1.0, 1.0), 1.0)
    _, ref_terms, ref = LF.loss_and_upstream([out], [tgt], (1.0, 1.0, 1.0), 1.0)
    l2 = rel_err(g[0][:3], ref[0][:3])[0]
    print(f"  {W}x{H}: gradient {l2:.2e}, 1 - SSIM {abs(terms[0, 1] - ref_terms[0][1]):.1e} off", flush=True)
    assert l2 <= TOL
