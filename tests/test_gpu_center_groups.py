"""Center selection by the packed 16-bit kernel (two centers and 64 partners per
group, strips of 32 rows) against the 32-bit kernel: the same integer sums at
the edges of groups, strips and column blocks, for odd candidate lists and for
gap costs up to what the packed kernel takes."""
import numpy as np
import pytest

from paper_1704_00878_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import paper_1704_00878_amd as H
    return H


@pytest.fixture(scope="module")
def ctx(H):
    c = H.Context(0)
    yield c
    c.close()


def _set(rng, n, lo, hi, empty=False):
    lens = rng.integers(lo, hi + 1, n)
    if empty:
        lens[rng.integers(0, n, 2)] = 0
    base = rng.integers(0, 20, hi).astype(np.uint8)
    seqs = []
    for L in lens:
        s = base[:L].copy()
        at = rng.random(L) < 0.4
        s[at] = rng.integers(0, 20, at.sum())
        seqs.append(s)
    return synth.SeqSet.from_list(seqs)


def _both(H, ctx, monkeypatch, run, n):
    import torch
    got = []
    for strip32 in ("0", "1"):
        monkeypatch.setenv("HALIGN_STRIP32", strip32)
        sums = torch.full((n,), -7, dtype=torch.int64, device="cuda")
        c = run(sums)
        got.append((c, sums.cpu()))
    assert got[0][0] == got[1][0] and bool((got[0][1] == got[1][1]).all())


@pytest.mark.parametrize("n", [2, 3, 63, 64, 65, 66, 127, 128, 129, 191, 192, 193, 450])
def test_exact_group_edges(H, ctx, n, monkeypatch):
    rng = np.random.default_rng(n)
    ds = H.DeviceSeqs(_set(rng, n, 1, 100, empty=n > 60))
    _both(H, ctx, monkeypatch, lambda s: H.halign_center_exact(ctx, H.Scoring(), ds, s), n)
    monkeypatch.setenv("HALIGN_GROUP_SLICE", "7")   # groups in sliced launches, from the last one down
    _both(H, ctx, monkeypatch, lambda s: H.halign_center_exact(ctx, H.Scoring(), ds, s), n)


# one strip and its neighbours, odd and even columns, and gap costs
@pytest.mark.parametrize("length", [1, 2, 3, 31, 32, 33, 64, 65, 97])
@pytest.mark.parametrize("go,ge", [(11, 1), (0, 1), (0, 50), (200, 56), (5, 38)])
def test_exact_strips_and_gaps(H, ctx, length, go, ge, monkeypatch):
    rng = np.random.default_rng(length)
    ds = H.DeviceSeqs(_set(rng, 70, max(1, length - 1), length))
    sc = H.Scoring(gap_open=go, gap_extend=ge)
    _both(H, ctx, monkeypatch, lambda s: H.halign_center_exact(ctx, sc, ds, s), 70)


# scores at the packed kernel's bound and past it
@pytest.mark.parametrize("length", [1355, 1361, 1362, 1363, 1364, 1370])
def test_exact_at_the_bound(H, ctx, length, monkeypatch):
    rng = np.random.default_rng(length)
    w = np.full(length, 17, np.uint8)   # W against W scores 11, the largest entry
    seqs = [w, w.copy(), w[:length - 1]] + [rng.integers(0, 20, length).astype(np.uint8) for _ in range(5)]
    seqs[4][100:900] = 17
    ds = H.DeviceSeqs(synth.SeqSet.from_list(seqs))
    _both(H, ctx, monkeypatch, lambda s: H.halign_center_exact(ctx, H.Scoring(), ds, s), len(seqs))


@pytest.mark.parametrize("cands", [1, 2, 3, 16, 17])
@pytest.mark.parametrize("partners", [0, 64, 131])
def test_judge_candidates(H, ctx, cands, partners, monkeypatch):
    import torch
    rng = np.random.default_rng(cands + partners)
    n = 201
    ds = H.DeviceSeqs(_set(rng, n, 20, 150))
    cand = torch.from_numpy(rng.permutation(n)[:cands].astype(np.int32)).cuda()
    part = rng.integers(0, n, partners).astype(np.int32)
    def run(s):
        if partners:
            return H.halign_center_judge_sample(ctx, H.Scoring(), ds, cand, part, s)
        return H.halign_center_judge(ctx, H.Scoring(), ds, cand, s)
    _both(H, ctx, monkeypatch, run, cands)
