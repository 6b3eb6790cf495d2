"""Pair emission in tiles of 8 on the widest frame: boxes of up to 256 tiles in a
row, of every width in between, wide, tall and square.  The forward's images do
not depend on the tile size, so a pair in a wrong tile shows."""
import numpy as np
import pytest

import scenes
from parity import gpu_params, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2511_16144_amd as P
    c = P.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("W,H", [(2048, 40), (72, 2048), (2041, 2047)])
def test_tile_sizes_agree(ctx, W, H):
    import paper_2511_16144_amd as P
    r = np.random.Generator(np.random.PCG64(W))
    n, f, z = 300, 500.0, 2.0
    # half-widths of 1 .. 1024 px across and 1 .. 1024 down, three sigmas each
    sx, sy = (np.exp(r.uniform(0, np.log(min(d, 2048) / 2), n)) / 3 * z / f for d in (W, H))
    u, v = r.uniform(0, W, n), r.uniform(0, H, n)
    cx, cy = (W - 1) / 2.0, (H - 1) / 2.0
    means = np.stack([(u - cx) * z / f, (v - cy) * z / f, z + 0.001 * np.arange(n)], 1).astype(np.float32)
    ls = np.log(np.stack([sx, sy, np.full(n, 1e-3)], 1)).astype(np.float32)
    feat = r.normal(size=(n, 16)).astype(np.float32)
    sc = scenes.Scene(means, ls, np.tile(np.float32([1, 0, 0, 0]), (n, 1)), r.normal(-2, 1, n).astype(np.float32),
                      r.uniform(0, 1, (n, 3)).astype(np.float32), feat, "f32")
    cams = [scenes.Camera(W, H, f, f, cx, cy, np.eye(3, dtype=np.float32), np.zeros(3, np.float32))]
    prm, res, pairs = gpu_params(sc), [], []
    for tile in (8, 16, 32):
        outs, state = ctx.forward(prm, cams, P.Settings(tile=tile), want_n=True)
        pairs.append(state.counts()["n_pairs"])
        res.append(to_np(outs)[0])
        state.release()
    print(f"  {W}x{H}: {pairs} pairs, up to {int(res[0]['n'].max())} contributors", flush=True)
    assert pairs[0] > pairs[1] > pairs[2] > n
    for other in res[1:]:
        for k in res[0]:
            assert np.array_equal(res[0][k], other[k]), k
