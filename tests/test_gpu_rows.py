"""Row emission against rows built in numpy, bytes compared: centers around the
prefetched words and both parities, empty rows, blocks placed by a lane and
by the whole wavefront, rows longer than what is staged, and widths of several
column chunks with blocks across their borders."""
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


def _case(rng, m, nrows, ends, wide):
    """Insertion counts (most 0, a few up to 9, the two ends up to `ends`, one
    block of `wide`), aligned bits, and the sequences they imply."""
    ins = np.where(rng.random((nrows, m + 1)) < 0.05, rng.integers(1, 10, (nrows, m + 1)), 0)
    ins[:, 0] = rng.integers(0, ends + 1, nrows)
    ins[:, m] = rng.integers(0, ends + 1, nrows)
    if wide:
        ins[rng.integers(0, nrows), m // 2] = wide
    al = (rng.random((nrows, m)) < 0.8).astype(np.uint8)
    ins[0], al[0] = 0, 0                       # an empty row
    ins[1], al[1] = 0, 1                       # the center itself
    n = ins.sum(1) + al.sum(1)
    return ins.astype(np.uint16), al, [rng.integers(0, 20, int(L)).astype(np.uint8) for L in n]


def _rows(ins, al, seqs, G, col, W):
    out = np.full((len(seqs), W), 255, np.uint8)
    for k, s in enumerate(seqs):
        q = 0
        for p in np.flatnonzero(ins[k] + np.append(al[k], 0)):
            c = int(ins[k, p])
            out[k, col[p]:col[p] + c] = s[q:q + c]
            q += c
            if p < al.shape[1] and al[k, p]:
                out[k, col[p] + G[p]] = s[q]
                q += 1
    return out


@pytest.mark.parametrize("m,nrows,ends,wide", [
    (1, 9, 3, 0), (2, 9, 0, 0), (31, 40, 60, 0), (63, 40, 5, 0), (64, 2100, 300, 0), (311, 3000, 200, 0), (510, 70, 9, 0),
    (511, 70, 9, 0), (512, 70, 9, 0), (1023, 20, 900, 0), (2047, 20, 40, 0), (2100, 20, 40, 0), (4000, 9, 3000, 0),
    (300, 30, 40, 20000), (5, 12, 17000, 9000), (1500, 30, 100, 8192)])
def test_rows(H, ctx, m, nrows, ends, wide, monkeypatch):
    import torch
    monkeypatch.setenv("HALIGN_ROWS", "lds")
    rng = np.random.default_rng(m + nrows)
    ins, al, seqs = _case(rng, m, nrows, ends, wide)
    aw = (m + 31) // 32
    words = np.zeros((nrows, aw), np.uint32)
    for p in range(m):
        words[:, p // 32] |= al[:, p].astype(np.uint32) << np.uint32(p % 32)
    G = ins.max(0).astype(np.int32)
    col = np.concatenate([[0], np.cumsum(G[:-1].astype(np.int64) + 1)])
    W = int(m + G.sum())
    ds = H.DeviceSeqs(synth.SeqSet.from_list(seqs))
    msa = torch.full((nrows, W), 77, dtype=torch.uint8, device="cuda")
    H.halign_emit_rows(ctx, ds, m, torch.from_numpy(ins.view(np.int16)).cuda(), torch.from_numpy(words.view(np.int32)).cuda(),
                       torch.from_numpy(G).cuda(), torch.from_numpy(col).cuda(), W, msa)
    assert (msa.cpu().numpy() == _rows(ins, al, seqs, G, col, W)).all()
