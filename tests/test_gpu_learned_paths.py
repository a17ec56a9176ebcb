"""The pipelined products of the learned center against the general ones.

The pipelined kernels (16-byte rows) and the general kernel (any alignment)
accumulate over k in the same order with the same matrix instruction, so their
results are the same bits: the same inputs are run once aligned and once from
buffers shifted by one element.  Top-k is compared with a stable sort."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import paper_1704_00878_amd as H
    H.lib()
    return H


@pytest.fixture(scope="module")
def ctx(H):
    c = H.Context(0)
    yield c
    c.close()


def shifted(t):
    """A copy of t that starts two bytes past a 16-byte boundary."""
    import torch
    b = torch.empty(t.numel() + 8, dtype=t.dtype, device=t.device)
    v = b[1:1 + t.numel()].view(t.shape)
    v.copy_(t)
    assert v.data_ptr() % 16 != 0
    return v


# both sides of each tile's edge (32 and 64 rows) and of each step of the rule
# on rows (a workgroup per CU: 2,048, 4,096 and 8,192 rows on 256 CUs)
@pytest.mark.parametrize("nrows", [1, 31, 33, 64, 2048, 2049, 4097, 8193])
def test_forward_same_bits(H, ctx, nrows):
    import torch
    g = torch.Generator("cuda").manual_seed(nrows)
    X = (torch.rand(nrows, H.FEAT, generator=g, device="cuda") * 3).floor().to(torch.bfloat16).view(torch.int16)
    prop = H.Proposer(seed=4)
    prop.b1.uniform_(-0.1, 0.1, generator=g)
    out = []
    for x, hb in ((X, torch.zeros(nrows, H.HID, dtype=torch.int16, device="cuda")),
                  (shifted(X), shifted(torch.zeros(nrows, H.HID, dtype=torch.int16, device="cuda")))):
        Z = torch.zeros(nrows, H.HID, device="cuda")
        E = torch.zeros(nrows, H.EMB, device="cuda")
        H.halign_mlp_forward(ctx, prop, x, nrows, Z, hb, E)
        out.append((Z, hb, E))
    for a, b in zip(*out):
        assert torch.equal(a, b)


# rows below, at and beyond a slice of 64 k (the contraction of the weight
# gradients runs over the rows), odd ones among them
@pytest.mark.parametrize("nrows", [1, 2, 63, 64, 65, 130, 1025])
def test_backward_same_bits(H, ctx, nrows):
    import torch
    g = torch.Generator("cuda").manual_seed(nrows)
    X = (torch.rand(nrows, H.FEAT, generator=g, device="cuda") * 3).floor().to(torch.bfloat16).view(torch.int16)
    Z = torch.randn(nrows, H.HID, generator=g, device="cuda")
    Hb = Z.clamp_min(0).to(torch.bfloat16).view(torch.int16)
    dE = torch.randn(nrows, H.EMB, generator=g, device="cuda")
    prop = H.Proposer(seed=4)
    out = []
    for x, hb in ((X, Hb), (shifted(X), shifted(Hb))):
        grads = [torch.full(s, 7.0, device="cuda") for s in ((H.FEAT, H.HID), (H.HID,), (H.HID, H.EMB), (H.EMB,))]
        H.halign_mlp_backward(ctx, prop, x, nrows, Z, hb, dE, *grads)
        out.append(grads)
    for a, b in zip(*out):
        assert torch.equal(a, b)
    # the bias gradients are plain sums of fp32 values: a fixed-order sum of n
    # terms is within n * 2^-24 of the sum of magnitudes
    ref = dE.double().sum(0)
    assert (out[0][3].double() - ref).abs().max() <= nrows * 2.0 ** -24 * dE.double().abs().sum(0).max()


@pytest.mark.parametrize("n,k", [(1, 1), (300, 256), (4096, 16), (4097, 16), (20000, 256)])
def test_topk_order(H, ctx, n, k):
    """Largest u first, ties (planted duplicates) to the lower index."""
    import torch
    g = torch.Generator("cuda").manual_seed(n)
    E = torch.randn(n, H.EMB, generator=g, device="cuda")
    E[n // 2:] = E[:n - n // 2].clone()
    u = torch.empty(n, device="cuda")
    top = torch.empty(k, dtype=torch.int32, device="cuda")
    H.halign_topk_center(ctx, E, n, k, u, top)
    want = np.argsort(-u.cpu().numpy(), kind="stable")[:k]
    assert (top.cpu().numpy() == want).all()
