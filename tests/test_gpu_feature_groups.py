"""Feature groups of 16 channels composited at once: a D-channel backward against
D / 16 backwards of 16 channels each, which take the same sums group by group.
The feature and colour gradients come out bit for bit; the geometric ones are
sums over the groups in another order (FP32, here of up to 8 terms: 1e-6
relative, 20 times that allowed for cancellation).  The large frame's records
pass 2 GB, so that its groups run in two batches, the second with the first
group in it."""
import numpy as np
import pytest
import torch

import scenes
from parity import gpu_params

pytestmark = pytest.mark.gpu
TOL = 2e-5


@pytest.fixture(scope="module")
def ctx():
    import paper_2511_16144_amd as P
    c = P.Context(0)
    yield c
    c.close()


SMALL = [(300, 61, 43, 32, 0), (300, 61, 43, 48, 2), (500, 96, 64, 128, 0)]


@pytest.mark.parametrize("n,w,h,D,covering,dtype", [(*c, d) for c in SMALL for d in ("f32", "bf16")] +
                         [(64, 1608, 1600, 128, 60, "bf16")])
def test_groups(ctx, n, w, h, D, covering, dtype):
    import paper_2511_16144_amd as P
    print(f"[case] {n} {w} x {h} D={D} {dtype}", flush=True)
    wl = scenes.tiny_scene(n + w, n, w, h, z_range=(1.0, 1.6), log_scale=(-2.5, 0.5))
    sc = wl.scene
    sc.logits = np.full(n, -2.0, np.float32)
    sc.log_scales[:covering] = np.float32([3.0, 3.1, 3.2])
    rng = np.random.default_rng(D)
    sc.feat = rng.standard_normal((n, D)).astype(np.float32)
    if dtype == "bf16":
        sc.rgb, sc.feat, sc.dtype = scenes.round_bf16(sc.rgb), scenes.round_bf16(sc.feat), "bf16"
    gen = torch.Generator(device="cuda").manual_seed(D)

    def up(c):
        return torch.randn((c, h, w), generator=gen, device="cuda")

    full = {"rgb": up(3), "depth": up(1)[0], "feat": up(D), "T": up(1)[0]}
    prm = gpu_params(sc)
    feat = prm["feat"]
    outs, state = ctx.forward(prm, wl.cams, P.Settings())
    if covering == 60:
        assert state.counts()["n_slots"] * 128 * (D // 16) > 2 ** 31
    for _ in range(2):   # the second over records and marks that the first left
        g = ctx.backward(state, prm, [full])
    torch.cuda.synchronize()
    state.release()
    images = outs[0]["feat"]
    total = {}
    for gi in range(D // 16):
        sl = slice(16 * gi, 16 * gi + 16)
        p16 = {**prm, "feat": feat[sl].contiguous()}
        o16, st16 = ctx.forward(p16, wl.cams, P.Settings())
        u = {k: (v if gi == 0 else torch.zeros_like(v)) for k, v in full.items()}
        u["feat"] = full["feat"][sl].contiguous()
        g16 = ctx.backward(st16, p16, [u])
        torch.cuda.synchronize()
        st16.release()
        assert torch.equal(o16[0]["feat"], images[sl])
        assert torch.equal(g16["feat"], g["feat"][sl])
        if gi == 0:
            assert torch.equal(o16[0]["rgb"], outs[0]["rgb"]) and torch.equal(o16[0]["T"], outs[0]["T"])
            assert torch.equal(g16["rgb"], g["rgb"])
        for k in ("means", "log_scales", "quats", "logits", "twist"):
            total[k] = total.get(k, 0.0) + g16[k].double()
    for k, t in total.items():
        err = float((g[k].double() - t).norm() / t.norm())
        print(f"  {k}: {err:.2e}", flush=True)
        assert err <= TOL, (k, err)
