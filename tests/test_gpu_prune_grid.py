"""Pruning where its table and lists change form, bit for bit against the FP64
pruning oracle: scenes of one cell up to the whole range of cells (2^20 to each
side), so that near and far cells fold onto the same buckets and runs go past
the table's end, with and without Gaussians that have no cell; knots of
k - 1 .. k + 2 neighbours (the last count taken as it is, the first that needs
an order); counts around the four-wide passes of the mask, the 64-wide ones of
the search and the powers of two of the table; 8 feature planes; a mask at an
odd address; a mean out of range, which leaves the mask as it was.
"""
import numpy as np
import pytest
import torch

from parity import gpu_params
from test_gpu_prune import check, ctx, make, run_both  # noqa: F401  (ctx: the fixture)

pytestmark = pytest.mark.gpu
TAU = 0.02


@pytest.mark.parametrize("bits", [(0, 0, 0), (1, 0, 2), (3, 3, 2), (7, 8, 9), (14, 13, 2), (20, 20, 20)])
@pytest.mark.parametrize("k,bf16,invalid", [(1, False, 0), (4, True, 3), (32, False, 1)])
def test_spans(ctx, bits, k, bf16, invalid):  # noqa: F811
    rng = np.random.default_rng(1000 * sum(bits) + k)
    side = TAU * (2.0 ** np.array(bits))      # cells per axis: 2^bits
    low = -np.floor(np.array([0.3, 0.5, 0.7]) * (2.0 ** np.array(bits))) * TAU
    P = [low + 0.25 * TAU, low + side - 0.25 * TAU]
    for c in ([0, 0, 0], [1, 1, 1], [0, 1, 0], [0.5, 0.5, 0.5], [0.3, 0.5, 0.7]):
        for m in (k, k + 1, k + 2, k + 3):    # k - 1 .. k + 2 neighbours each
            at = low + (0.5 + np.array(c) * (2.0 ** np.array(bits) - 1)) * TAU
            at = at + rng.uniform(-0.1, 0.1, 3) * TAU
            P.append(at + rng.uniform(-0.3, 0.3, (m, 3)) * TAU)
    P = np.concatenate([np.atleast_2d(p) for p in P])
    P = np.clip(P, low + 0.01 * TAU, low + side - 0.01 * TAU)
    n = len(P)
    base = rng.standard_normal((3, 16))
    F = base[rng.integers(0, 3, n)] + 0.1 * rng.standard_normal((n, 16))
    lam = rng.choice([-1.0, 0.0, 0.5, 2.0, -6.0], n)
    ls = np.full((n, 3), -4.0)
    bad = rng.permutation(n)[:invalid]
    P[bad, rng.integers(0, 3, len(bad))] = np.array([np.nan, np.inf, -np.inf])[:len(bad)]
    sc = make(P, F, lam, ls, bf16)
    check(f"bits {bits} k {k} bf16 {bf16} invalid {invalid}", sc, *run_both(ctx, sc, k=k, tau_dist=TAU), tau_dist=TAU)


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 63, 64, 65, 127, 128, 129, 1023, 1024, 1025])
@pytest.mark.parametrize("spread", [0.05, 3.0])
def test_counts(ctx, n, spread):  # noqa: F811
    rng = np.random.default_rng(n)
    P = rng.uniform(-spread, spread, (max(1, n // 4), 3))[rng.integers(0, max(1, n // 4), n)]
    P = P + rng.uniform(-0.008, 0.008, (n, 3))
    F = rng.standard_normal((3, 16))[rng.integers(0, 3, n)]
    sc = make(P, F, rng.choice([-6.0, 0.0, 1.0], n), rng.choice([-4.0, 0.0], (n, 3)))
    check(f"n {n}", sc, *run_both(ctx, sc, k=4, tau_dist=TAU), tau_dist=TAU)


def test_none_has_a_cell(ctx):  # noqa: F811
    sc = make(np.full((70, 3), np.nan), np.ones((70, 16)), np.zeros(70), np.full((70, 3), -4.0))
    check("no cell", sc, *run_both(ctx, sc))


@pytest.mark.parametrize("bf16", [False, True])
def test_eight_planes_and_odd_mask(ctx, bf16):  # noqa: F811
    rng = np.random.default_rng(8)
    n = 301
    P = rng.uniform(-0.05, 0.05, (n, 3))
    F = rng.standard_normal((3, 16))[rng.integers(0, 3, n)] + 0.3 * rng.standard_normal((n, 16))
    F[:, 8:] = 0.0
    sc = make(P, F, rng.choice([-6.0, 0.0, 1.0], n), np.full((n, 3), -4.0), bf16)
    m, counts, *rest = run_both(ctx, sc, k=8, tau_dist=TAU)
    check(f"16 planes bf16 {bf16}", sc, m, counts, *rest)
    g = dict(gpu_params(sc))
    g["feat"] = g["feat"][:8].contiguous()
    buf = torch.full((n + 8,), 255, dtype=torch.uint8, device="cuda")
    prm = dict(k=8, tau_dist=float(np.float32(TAU)), tau_sim=float(np.float32(0.9)),
               min_opacity=float(np.float32(0.005)), max_scale=float(np.float32(0.3)))
    for at in (1, 2, 3, 4):
        buf.fill_(255)
        _, c8 = ctx.prune(g, mask=buf[at:at + n], **prm)
        assert c8 == counts and np.array_equal(buf[at:at + n].cpu().numpy(), m)
        assert bool((buf[:at] == 255).all()) and bool((buf[at + n:] == 255).all())


def test_out_of_range_leaves_the_mask(ctx):  # noqa: F811
    P = np.zeros((5, 3))
    P[3, 1] = 2.0 ** 20 * TAU * 1.01
    sc = make(P, np.ones((5, 16)), np.zeros(5), np.full((5, 3), -4.0))
    buf = torch.full((5,), 77, dtype=torch.uint8, device="cuda")
    with pytest.raises(Exception):
        ctx.prune(gpu_params(sc), mask=buf, tau_dist=TAU)
    assert bool((buf == 77).all())
    P[3, 1] = 0.0
    sc = make(P, np.ones((5, 16)), np.zeros(5), np.full((5, 3), -4.0))
    check("after the error", sc, *run_both(ctx, sc))
