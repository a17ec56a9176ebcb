"""Alphabets up to the largest (32 codes, none left for padding) on every kernel,
against the oracle: sequences of different lengths side by side, whose padding
columns must not score, with matrices in which the last codes score best."""
import numpy as np
import pytest

import oracle
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


def _set(alpha, n=90):
    rng = np.random.default_rng(alpha)
    mat = rng.integers(-6, 4, (alpha, alpha)).astype(np.int8)
    mat = np.minimum(mat, mat.T)
    mat[alpha - 1] = mat[:, alpha - 1] = 3      # the last code fits every other
    np.fill_diagonal(mat, 5)
    lens = np.concatenate([rng.integers(0, 150, n - 2), [1, 260]])
    return mat, [rng.integers(0, alpha, int(L)).astype(np.uint8) for L in lens]


def _want(mat, seqs, center, go, ge):
    return [oracle.sw(mat, go, ge, center, s) for s in seqs]


KNOBS = {"default": {}, "strip": {"HALIGN_ROUTE": "inter"}, "lanes64": {"HALIGN_STREAM_LANES": "64"},
         "profile32": {"HALIGN_PROFILE32": "1", "HALIGN_ROUTE": "intra"},
         "lanes16": {"HALIGN_STREAM_LANES": "16", "HALIGN_STREAM_PACK": "0"},
         "packed": {"HALIGN_STREAM_LANES": "32", "HALIGN_STREAM_PACK": "1"}}


@pytest.mark.parametrize("knobs", list(KNOBS))
@pytest.mark.parametrize("m", [40, 600])
@pytest.mark.parametrize("alpha", [1, 2, 24, 31, 32])
def test_batch(H, ctx, alpha, m, knobs, monkeypatch):
    import torch
    for k, v in KNOBS[knobs].items():
        monkeypatch.setenv(k, v)
    if alpha == 1:
        mat, seqs = np.full((1, 1), 2, np.int8), [np.zeros(int(L), np.uint8) for L in range(0, 90)]
    else:
        mat, seqs = _set(alpha)
    center = np.random.default_rng(m).integers(0, alpha, m).astype(np.uint8)
    want = _want(mat, seqs, center, 4, 1)
    ds = H.DeviceSeqs(synth.SeqSet.from_list(seqs))
    for tb in (False, True):
        out = H.sw_batch(ctx, H.Scoring(mat, 4, 1), ds, 0, traceback=tb, center_seq=torch.from_numpy(center).cuda())
        assert (out["score"].cpu().numpy() == [w["score"] for w in want]).all()
        first = 0 if tb else 2      # score-only calls give the end cell alone
        cells = np.stack([w["cells"] for w in want])
        assert (out["cells"].cpu().numpy()[:, first:] == cells[:, first:]).all()


@pytest.mark.parametrize("strip32", ["0", "1"])
@pytest.mark.parametrize("alpha", [2, 24, 31, 32])
def test_centers(H, ctx, alpha, strip32, monkeypatch):
    import torch
    monkeypatch.setenv("HALIGN_STRIP32", strip32)
    mat, seqs = _set(alpha, 70)
    n = len(seqs)
    M = np.zeros((n, n), np.int64)
    for a in range(n):
        for b in range(a + 1, n):
            M[a, b] = M[b, a] = oracle.sw(mat, 4, 1, seqs[a], seqs[b])["score"]
    ds = H.DeviceSeqs(synth.SeqSet.from_list(seqs))
    sums = torch.empty(n, dtype=torch.int64, device="cuda")
    c = H.halign_center_exact(ctx, H.Scoring(mat, 4, 1), ds, sums)
    assert (sums.cpu().numpy() == M.sum(1)).all() and c == int(M.sum(1).argmax())
    cand = torch.tensor([3, n - 1, 7], dtype=torch.int32, device="cuda")
    got = torch.empty(3, dtype=torch.int64, device="cuda")
    H.halign_center_judge(ctx, H.Scoring(mat, 4, 1), ds, cand, got)
    assert (got.cpu().numpy() == M.sum(1)[[3, n - 1, 7]]).all()


@pytest.mark.parametrize("alpha", [2, 31, 32])
def test_scores_without_a_context(H, alpha):
    import torch
    mat, seqs = _set(alpha)
    center = np.random.default_rng(3).integers(0, alpha, 90).astype(np.uint8)
    want = _want(mat, seqs, center, 4, 1)
    ds = H.DeviceSeqs(synth.SeqSet.from_list(seqs))
    score = torch.empty(len(seqs), dtype=torch.int32, device="cuda")
    H.halign_sw_score_noalloc(H.Scoring(mat, 4, 1), torch.from_numpy(center).cuda(), 90, ds, score)
    torch.cuda.synchronize()
    assert (score.cpu().numpy() == [w["score"] for w in want]).all()
