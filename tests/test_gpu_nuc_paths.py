"""The nucleotide path where its kernels change form: the segment table's sizes
and repeats, both scans, chains in LDS and in global arrays, stretches settled
on the diagonal or by the dynamic program on a lane or a wavefront, and lists
that outgrow their first guess.  Scores and center-star vectors against the
oracle, bit for bit."""
import numpy as np
import pytest

import oracle
from paper_1704_00878_amd import synth

pytestmark = pytest.mark.gpu
NM, GO, GE = synth.NUC_MATRIX, synth.NUC_GAP_OPEN, synth.NUC_GAP_EXTEND


@pytest.fixture(scope="module")
def H():
    import paper_1704_00878_amd as H
    return H


def _check(H, ctx, seqs, k, mat=NM, go=GO, ge=GE, center=0):
    import torch
    seqs = synth.SeqSet.from_list([np.asarray(s, np.uint8) for s in seqs])
    N, c = seqs.n, seqs.seq(center)
    m = len(c)
    score = torch.empty(N, dtype=torch.int32, device="cuda")
    ins = torch.empty((N, m + 1), dtype=torch.int16, device="cuda")
    al = torch.empty((N, (m + 31) // 32), dtype=torch.int32, device="cuda")
    G = torch.empty(m + 1, dtype=torch.int32, device="cuda")
    H.halign_nuc_align(ctx, H.Scoring(mat, go, ge), H.DeviceSeqs(seqs), center, k, score, ins, al, G)
    torch.cuda.synchronize()
    words = al.cpu().numpy().view(np.uint32)
    bits = ((words[:, :, None] >> np.arange(32, dtype=np.uint32)) & 1).reshape(N, -1)[:, :m]
    ins = ins.cpu().numpy().view(np.uint16)
    want = [oracle.nuc_align(mat, go, ge, k, c, seqs.seq(x)) for x in range(N)]
    assert (score.cpu().numpy() == [w["score"] for w in want]).all()
    assert (ins == np.stack([w["ins"] for w in want])).all()
    assert (bits == np.stack([w["aligned"] for w in want])).all()
    assert (G.cpu().numpy() == np.delete(ins, center, 0).max(0)).all()


def _mutate(rng, c, p_sub, p_indel):
    s = c.copy()
    at = rng.random(len(s)) < p_sub
    s[at] = (s[at] + rng.integers(1, 4, at.sum())) % 4
    out = []
    for i, b in enumerate(s):
        r = rng.random()
        if r < p_indel:
            continue
        out.append(b)
        if r > 1 - p_indel:
            out.extend(rng.integers(0, 4, rng.integers(1, 6)))
    return np.array(out, np.uint8)


# every string repeated; tables at and past the LDS size; 32- and 64-bit keys; both
# scans; the center not a multiple of k
@pytest.mark.parametrize("k,m", [(1, 300), (2, 301), (3, 1000), (4, 3000), (6, 13000), (16, 33000), (17, 3000), (29, 2000),
                                 (30, 2000), (32, 2031), (16, 15), (16, 16)])
def test_segments(H, k, m):
    ctx = H.Context(0)
    rng = np.random.default_rng(k * 7 + m)
    c = rng.integers(0, 4, m).astype(np.uint8)
    if m > 100:
        c[m // 2:m // 2 + 40] = c[:40]
        c[m // 3] = 4
    _check(H, ctx, [c, _mutate(rng, c, 0.01, 0.002), _mutate(rng, c, 0.05, 0.01), c[m // 4:], c[:0]], k)
    ctx.close()


# few anchors fit the center, but long sequences match it thousands of times
@pytest.mark.parametrize("n", [300, 9000, 30000])
def test_many_matches(H, n):
    ctx = H.Context(0)
    rng = np.random.default_rng(n)
    c = rng.integers(0, 4, 500).astype(np.uint8)
    _check(H, ctx, [c, rng.integers(0, 4, n), _mutate(rng, c, 0.02, 0.01), rng.integers(0, 4, n // 2)], 4)
    ctx.close()


# the diagonal's bound from both sides: 0 .. 6 substitutions in stretches of one,
# two and three segments, and in one that is longer than a lane tests
@pytest.mark.parametrize("lanes", ["0", "1000000"])
@pytest.mark.parametrize("go,ge", [(5, 2), (0, 1), (1, 1), (40, 3)])
def test_diagonal(H, lanes, go, ge, monkeypatch):
    monkeypatch.setenv("HALIGN_NUC_LANES", lanes)
    ctx = H.Context(0)
    rng = np.random.default_rng(go)
    c = rng.integers(0, 4, 900).astype(np.uint8)
    c[320:480] = np.tile(c[:16], 10)    # not indexed: a stretch of 160
    seqs = [c]
    for span in (14, 30, 46):
        for nsub in range(7):
            s = c.copy()
            at = 161 + rng.permutation(span)[:nsub]
            s[at] = (s[at] + rng.integers(1, 4, nsub)) % 4
            s[330 + rng.permutation(140)[:nsub]] = 4
            seqs.append(s)
    _check(H, ctx, seqs, 16, go=go, ge=ge)
    ctx.close()


# matrices with ties and with rows that have no positive score
@pytest.mark.parametrize("lanes", ["0", "1000000"])
@pytest.mark.parametrize("seed", range(6))
def test_matrices(H, lanes, seed, monkeypatch):
    monkeypatch.setenv("HALIGN_NUC_LANES", lanes)
    ctx = H.Context(0)
    rng = np.random.default_rng(seed)
    mat = rng.integers(-3, 3, (5, 5)).astype(np.int8)
    mat = np.minimum(mat, mat.T)
    c = rng.integers(0, 4, 1500).astype(np.uint8)
    _check(H, ctx, [c] + [_mutate(rng, c, 0.02, 0.004) for _ in range(12)], 8, mat, int(rng.integers(0, 4)),
           int(rng.integers(1, 3)))
    ctx.close()


# lists, codes and boundary columns past their first guess, then a small call
# on the grown buffers
@pytest.mark.parametrize("lanes", ["0", "1000000"])
def test_lists_grow(H, lanes, monkeypatch):
    monkeypatch.setenv("HALIGN_NUC_LANES", lanes)
    ctx = H.Context(0)
    rng = np.random.default_rng(4)
    c = rng.integers(0, 4, 20000).astype(np.uint8)
    _check(H, ctx, [c] + [_mutate(rng, c, 0.06, 0.02) for _ in range(9)] + [rng.integers(0, 4, 900)], 8)
    _check(H, ctx, [c[:700], _mutate(rng, c[:700], 0.01, 0.01)], 16)
    ctx.close()


def test_bad_code_refused(H):
    ctx = H.Context(0)
    rng = np.random.default_rng(8)
    seqs = [rng.integers(0, 4, 400).astype(np.uint8) for _ in range(3)]
    seqs[1][77] = 9
    with pytest.raises(H.HalignError):
        _check(H, ctx, seqs, 16)
    seqs[1][77] = 4
    _check(H, ctx, seqs, 16)
    ctx.close()


# column sums and chunked rows around their tiles (4,096 positions; 256 blocks a
# chunk, four chunks in flight on each of four wavefronts) and parities
@pytest.mark.parametrize("m", [254, 255, 256, 4094, 4095, 4096, 4097, 8191, 16639, 65535])
def test_merge_and_chunked_rows(H, m, monkeypatch):
    monkeypatch.setenv("HALIGN_ROWS", "chunk")
    ctx = H.Context(0)
    rng = np.random.default_rng(m)
    c = rng.integers(0, 4, m).astype(np.uint8)
    seqs = synth.SeqSet.from_list([c] + [_mutate(rng, c, 0.002, 0.0005)[:65535] for _ in range(4)])
    ref = oracle.nuc_msa(NM, GO, GE, 16, seqs.residues, seqs.offsets)
    msa, score = H.halign_nuc_msa(ctx, H.Scoring(NM, GO, GE), H.DeviceSeqs(seqs), 16)
    assert msa.shape[1] == ref["width"]
    assert (msa.cpu().numpy() == ref["msa"]).all() and (score.cpu().numpy() == ref["score"]).all()
    ctx.close()
