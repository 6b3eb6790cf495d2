"""The pair emission divides a pair's place in its Gaussian's tile box by the
box's width through a reciprocal of about 1 ulp: every place (at most 2^16
tiles) and width, with the reciprocal off by up to 2 ulps either way, in FP32
as the kernel computes it."""
import numpy as np
import pytest


@pytest.mark.parametrize("ulps", [-2, -1, 0, 1, 2])
def test_quotient_is_exact(ulps):
    local = np.arange(1 << 16, dtype=np.uint32)
    x = local.astype(np.float32) + np.float32(0.5)
    for w in range(1, 257):
        r = (np.float32(1.0) / np.float32(w)).view(np.int32) + np.int32(ulps)
        q = (x * r.view(np.float32)).astype(np.uint32)
        assert np.array_equal(q, local // w), w
