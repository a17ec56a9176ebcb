"""Joins that the mesh of workgroups leaves to the other kernels: the tree is
theirs, bit for bit."""
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


# distances that are infinite or NaN, one pair of them or many, in problems that
# go to one workgroup (up to 256 nodes) and to the whole chip otherwise; sums that overflow
@pytest.mark.parametrize("share", [0.0, 0.1])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 1.5e308])
@pytest.mark.parametrize("n", [8, 40, 256, 300])
def test_not_finite(H, ctx, n, value, share, monkeypatch):
    import torch
    rng = np.random.default_rng(n)
    d = np.triu(rng.random((n, n)), 1)
    d[np.triu(rng.random((n, n)) < share, 1)] = value
    d[2, 3:5] = value
    D = torch.from_numpy(np.triu(d, 1) + np.triu(d, 1).T).cuda()
    got = H.halign_nj(ctx, D)
    monkeypatch.setenv("HALIGN_NJ_MESH", "0")
    want = H.halign_nj(ctx, D)
    assert len(got[0]) == len(want[0])
    assert (got[0] == want[0]).all() and (got[1].view(np.int64) == want[1].view(np.int64)).all()


# waits that give up at once or after a few polls (some workgroups may get
# further than others before they see it), alone and in a tree with small
# clusters on the second stream; the context serves a problem that the mesh finishes afterwards
@pytest.mark.parametrize("spin", ["0", "1", "3"])
@pytest.mark.parametrize("n", [8, 17, 256, 257, 700])
def test_gives_up(H, ctx, n, spin, monkeypatch):
    import torch
    rng = np.random.default_rng(n)
    d = np.triu(rng.random((n, n)), 1)
    D = torch.from_numpy(d + d.T).cuda()
    keep = D.clone()
    monkeypatch.setenv("HALIGN_NJ_MESH", "0")
    want = H.halign_nj(ctx, D)
    monkeypatch.delenv("HALIGN_NJ_MESH")
    monkeypatch.setenv("HALIGN_NJ_SPIN", spin)
    got = H.halign_nj(ctx, D)
    monkeypatch.delenv("HALIGN_NJ_SPIN")
    after = H.halign_nj(ctx, D)
    assert torch.equal(D, keep)
    for x in (got, after):
        assert (x[0] == want[0]).all() and (x[1].view(np.int64) == want[1].view(np.int64)).all()


@pytest.mark.parametrize("full", ["1", "0"])
def test_tree_gives_up(H, ctx, full, monkeypatch):
    import torch
    rng = np.random.default_rng(4)
    n, w = 400, 500
    root = rng.integers(0, 4, w)
    m = np.where(rng.random((n, w)) < 0.02, rng.integers(0, 4, (n, w)), root).astype(np.uint8)
    dev = torch.from_numpy(m).cuda()
    perm = rng.permutation(n).astype(np.int32)
    monkeypatch.setenv("HALIGN_NJ_FULL", full)
    monkeypatch.setenv("HALIGN_NJ_MESH", "0")
    want = H.halign_nj_tree(ctx, dev, perm)
    monkeypatch.delenv("HALIGN_NJ_MESH")
    monkeypatch.setenv("HALIGN_NJ_SPIN", "0")
    got = H.halign_nj_tree(ctx, dev, perm)
    assert (got[0] == want[0]).all() and (got[1].view(np.int64) == want[1].view(np.int64)).all()
