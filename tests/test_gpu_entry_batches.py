"""The compositing kernels take a block's entries in pairs (forward) and in
groups of four and batches of sixteen (backward), each with a remainder.
Scenes in which every Gaussian reaches most of a 13 x 11 image, with entry
counts around those sizes and around a 64-entry chunk, against the FP64
oracle; features of one partial group (8 channels) and of one full one."""
import numpy as np
import pytest
import torch

import scenes
from oracle import raster_fp64 as R
from parity import (TOL_F32, ambiguous, forward_errors, fmt, gpu_params, grad_errors, grads_np, mask_upstream,
                    separate_targets, to_np, upstream_tensors)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2511_16144_amd as P
    c = P.Context(0)
    yield c
    c.close()


def workload(n, dtype, D):
    wl = scenes.tiny_scene(200 + n, n, 13, 11, z_range=(1.0, 1.6), log_scale=(-1.6, 0.2))
    sc = wl.scene
    rng = np.random.Generator(np.random.PCG64(n))
    sc.logits = rng.normal(-3.0, 0.4, size=n).astype(np.float32)   # no pixel ends before its last entry
    sc.feat = np.ascontiguousarray(sc.feat[:, :D])
    if dtype == "bf16":
        sc.rgb, sc.feat, sc.dtype = scenes.round_bf16(sc.rgb), scenes.round_bf16(sc.feat), "bf16"
    wl.targets = [scenes.Targets(t.rgb, t.depth, np.ascontiguousarray(t.feat[:D])) for t in wl.targets]
    return wl


@pytest.mark.parametrize("dtype,D", [("f32", 16), ("bf16", 16), ("bf16", 8)])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 15, 16, 17, 31, 33, 64, 65, 130])
def test_entry_counts(ctx, n, dtype, D):
    import paper_2511_16144_amd as P
    print(f"[case] {n} entries {dtype} D={D}", flush=True)
    wl = workload(n, dtype, D)
    ref = R.render(wl.scene, wl.cams, R.Settings())
    amb = ambiguous(ref[0]["margin"])
    prm = gpu_params(wl.scene)
    outs, state = ctx.forward(prm, wl.cams, P.Settings(), want_n=True)
    out = to_np(outs)[0]
    err = forward_errors(out, ref[0], amb)
    assert np.array_equal(out["n"][~amb], ref[0]["n"][~amb]) and out["n"].max() > n // 2
    # a given upstream, zero at the ambiguous pixels: every Gaussian compared
    ups = mask_upstream(scenes.random_upstream(n, wl.cams, feat_dim=D), [amb])
    g = grads_np(ctx.backward(state, prm, upstream_tensors(ups)))
    err.update({"given " + k: v for k, v in grad_errors(g, R.vjp(wl.scene, wl.cams, ups, R.Settings()),
                                                        np.zeros(n, bool)).items()})
    if not amb.any():
        # the fused L1 gradient, residuals kept off zero
        tg = separate_targets(ref, wl.targets)
        dev = [{k: torch.as_tensor(getattr(t, k)).cuda() for k in ("rgb", "depth", "feat")} for t in tg]
        g = grads_np(ctx.backward_l1(state, prm, outs, dev, (1.0, 0.5, 2.0)))
        hw = float(out["T"].size)
        u = np.concatenate([np.sign(ref[0]["rgb"] - tg[0].rgb) / (3 * hw),
                            0.5 * np.sign(ref[0]["depth"] - tg[0].depth)[None] / hw,
                            2.0 * np.sign(ref[0]["feat"] - tg[0].feat) / (D * hw)])
        err.update({"L1 " + k: v for k, v in grad_errors(g, R.vjp(wl.scene, wl.cams, [u], R.Settings()),
                                                         np.zeros(n, bool)).items()})
    torch.cuda.synchronize()
    state.release()
    print("  " + fmt(err), flush=True)
    for k, (l2, mx) in err.items():
        assert l2 <= TOL_F32 and mx <= TOL_F32, (k, l2, mx)
