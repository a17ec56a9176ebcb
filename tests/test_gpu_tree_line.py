"""Trees on both sides of the line between all distances at once and a launch per
step: the same bits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [767, 768, 769, 2048])
def test_same_tree(n, monkeypatch):
    import torch
    import paper_1704_00878_amd as H
    rng = np.random.default_rng(n)
    root = rng.integers(0, 4, 300)
    m = np.where(rng.random((n, 300)) < 0.05, rng.integers(0, 4, (n, 300)), root).astype(np.uint8)
    m[rng.random((n, 300)) < 0.05] = 255
    dev = torch.from_numpy(m).cuda()
    perm = rng.permutation(n).astype(np.int32)
    ctx = H.Context(0)
    got = H.halign_nj_tree(ctx, dev, perm)
    monkeypatch.setenv("HALIGN_NJ_FULL", "0")
    want = H.halign_nj_tree(ctx, dev, perm)
    ctx.close()
    assert (got[0] == want[0]).all() and (got[1].view(np.int64) == want[1].view(np.int64)).all()
