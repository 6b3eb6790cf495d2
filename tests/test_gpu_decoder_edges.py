"""The decoder loss at the edges of its chunks (32 pixels): sizes around one
chunk, runs of several chunks per work-group that end with and without a
partial one, and targets that start at any element.  Against the formula in
FP64 (targets at least 0.02 from the decoded values, so that every sign is the
same on both sides); 1e-4 relative to each output's norm, since the operands
carry 16 significant bits and the sums are FP32.  The same targets at another
alignment give the same bits.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu

SIZES = [1, 31, 32, 33, 71, 32 * 256 * 2, 32 * 256 * 2 + 7, 32 * 256 * 4 + 33]


@pytest.fixture(scope="module")
def ctx():
    import paper_2511_16144_amd as P
    c = P.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("C", [256, 512])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "f32"])
def test_chunk_edges(ctx, n, C, dtype):
    print(n, C, dtype, flush=True)
    g = torch.Generator(device="cuda").manual_seed(n + C)
    F = 0.25 * torch.randn(16, 1, n, device="cuda", generator=g)
    W = 0.25 * torch.randn(C, 16, device="cuda", generator=g)
    b = 0.05 * torch.randn(C, device="cuda", generator=g)
    Z = W.double() @ F.double().reshape(16, n) + b.double()[:, None]
    r = 0.3 * torch.randn(C, n, device="cuda", generator=g)
    T = (Z + r + torch.where(r >= 0, 0.05, -0.05)).to(dtype).reshape(C, 1, n)
    R = torch.sign(Z - T.reshape(C, n).double())
    s = 1.0 / (C * n)
    want = [s * (Z - T.reshape(C, n).double()).abs().sum(), s * W.double().t() @ R,
            s * R @ F.double().reshape(16, n).t(), s * R.sum(1)]
    assert float((Z - T.reshape(C, n).double()).abs().min()) > 0.02
    got = [x.clone() for x in ctx.decoder_l1(F, W, b, T)]
    for x, y in zip(got, want):
        d = x.double().reshape(y.shape) - y
        assert float(d.norm()) <= 1e-4 * float(y.norm()) + 1e-12
    for off in (1, 2, 3):
        shifted = torch.empty(C * n + off, dtype=dtype, device="cuda")[off:].reshape(C, 1, n)
        shifted.copy_(T)
        for x, y in zip(got, ctx.decoder_l1(F, W, b, shifted)):
            assert torch.equal(x, y)
