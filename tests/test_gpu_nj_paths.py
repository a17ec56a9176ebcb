"""The tree's faster paths against its general ones, bit for bit: neighbour
joining on a mesh of workgroups against the chip-wide kernels (the same double
operations in the same order), trees from all distances computed at once
against a launch per step, and distances of one triangle and of column slices
against whole row lists.  The general paths are compared with the oracle
elsewhere."""
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


# last workgroups of 1 and 16 rows, the largest problem of the mesh and the
# first beyond it; distances with many ties (small integers) and without
@pytest.mark.parametrize("ties", [False, True])
@pytest.mark.parametrize("n", [257, 272, 500, 1024, 1025])
def test_mesh_same_bits(H, ctx, n, ties, monkeypatch):
    import torch
    rng = np.random.default_rng(n)
    d = rng.integers(1, 5, (n, n)).astype(float) if ties else rng.random((n, n))
    d = np.triu(d, 1)
    D = torch.from_numpy(d + d.T).cuda()
    keep = D.clone()
    got = H.halign_nj(ctx, D)
    monkeypatch.setenv("HALIGN_NJ_MESH", "0")
    want = H.halign_nj(ctx, D)
    assert torch.equal(D, keep)
    assert (got[0] == want[0]).all() and (got[1].view(np.int64) == want[1].view(np.int64)).all()


# the smallest problems the mesh takes, one workgroup of 16 rows and two
@pytest.mark.parametrize("n", [8, 9, 16, 17, 33, 100, 256])
def test_mesh_small(H, ctx, n, monkeypatch):
    import torch
    rng = np.random.default_rng(n)
    d = np.triu(rng.random((n, n)), 1)
    D = torch.from_numpy(d + d.T).cuda()
    got = H.halign_nj(ctx, D)
    monkeypatch.setenv("HALIGN_NJ_MESH", "0")   # one workgroup
    want = H.halign_nj(ctx, D)
    assert (got[0] == want[0]).all() and (got[1].view(np.int64) == want[1].view(np.int64)).all()


# random rows (no structure), near-identical rows (many divide passes, runs of
# rows that one seed takes), all-gap rows, and few rows
@pytest.mark.parametrize("n,w,p,gaps", [(7, 40, 0.5, 0), (60, 200, 0.5, 3), (300, 900, 0.01, 0), (300, 900, 0.3, 5),
                                        (700, 300, 0.0, 0)])
def test_tree_from_all_distances(H, ctx, n, w, p, gaps, monkeypatch):
    import torch
    rng = np.random.default_rng(n + w)
    root = rng.integers(0, 4, w)
    m = np.where(rng.random((n, w)) < p, rng.integers(0, 4, (n, w)), root).astype(np.uint8)
    m[rng.random((n, w)) < 0.05] = 255
    m[:gaps] = 255
    dev = torch.from_numpy(m).cuda()
    perm = rng.permutation(n).astype(np.int32)
    got = H.halign_nj_tree(ctx, dev, perm)
    monkeypatch.setenv("HALIGN_NJ_FULL", "0")
    want = H.halign_nj_tree(ctx, dev, perm)
    assert (got[0] == want[0]).all() and (got[1].view(np.int64) == want[1].view(np.int64)).all()


# tile edges, one and several slices, widths that are no multiple of a slice
@pytest.mark.parametrize("n,w", [(1, 1), (63, 255), (64, 257), (65, 1000), (129, 4001), (200, 64)])
def test_pdist_one_triangle(H, ctx, n, w):
    import torch
    rng = np.random.default_rng(n + w)
    m = rng.integers(0, 20, (n, w)).astype(np.uint8)
    m[rng.random((n, w)) < 0.3] = 255
    dev = torch.from_numpy(m).cuda()
    ids = torch.arange(n, dtype=torch.int32, device="cuda")
    got = H.halign_pdist(ctx, dev, counts=True)
    same = H.halign_pdist(ctx, dev, ids, ids, counts=True)
    want = H.halign_pdist(ctx, dev, ids, ids.clone(), counts=True)   # two lists: every tile
    for a, b, c in zip(got, same, want):
        assert torch.equal(a, c) and torch.equal(b, c)
