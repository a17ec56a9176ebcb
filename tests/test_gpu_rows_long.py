"""Row emission for more center positions than a sequence can hold (vectors made
by a caller): 288 chunks of 256 blocks and one more, two tiles of 256 chunks and
one chunk more, and a ragged number, against rows built in numpy."""
import numpy as np
import pytest

from paper_1704_00878_amd import synth
from test_gpu_rows import _rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [65535, 65536, 73727, 73728, 131071, 131072, 200003])
def test_more_positions_than_a_sequence(m):
    import torch
    import paper_1704_00878_amd as H
    rng = np.random.default_rng(m)
    nrows = 5
    ins = np.where(rng.random((nrows, m + 1)) < 0.01, rng.integers(1, 10, (nrows, m + 1)), 0)
    al = (rng.random((nrows, m)) < 0.2).astype(np.uint8)
    ins[0], al[0] = 0, 0                       # an empty row
    ins[1, : m - 500], al[1, : m - 500] = 0, 0   # residues in the last chunks only
    n = ins.sum(1) + al.sum(1)
    seqs = [rng.integers(0, 20, int(L)).astype(np.uint8) for L in n]
    ins = ins.astype(np.uint16)
    bits = np.zeros((nrows, (m + 31) // 32 * 32), np.uint8)
    bits[:, :m] = al
    words = np.packbits(bits, axis=1, bitorder="little").view(np.int32)
    G = ins.max(0).astype(np.int32)
    col = np.concatenate([[0], np.cumsum(G[:-1].astype(np.int64) + 1)])
    W = int(m + G.sum())
    ctx = H.Context(0)
    ds = H.DeviceSeqs(synth.SeqSet.from_list(seqs))
    msa = torch.full((nrows, W), 77, dtype=torch.uint8, device="cuda")
    H.halign_emit_rows(ctx, ds, m, torch.from_numpy(ins.view(np.int16)).cuda(), torch.from_numpy(words).cuda(),
                       torch.from_numpy(G).cuda(), torch.from_numpy(col).cuda(), W, msa)
    assert (msa.cpu().numpy() == _rows(ins, al, seqs, G, col, W)).all()
    ctx.close()
