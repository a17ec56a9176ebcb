"""Plans that the library chooses by itself against the one-pair-per-lane
kernel: the same pairs give the same scores, end cells, insertion counts and
aligned bits on every plan (integers, compared exactly; the one-pair-per-lane
kernel is compared with the oracle elsewhere)."""
import numpy as np
import pytest

from paper_1704_00878_amd import synth

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


def _same(H, ctx, sc, ds, center, tb):
    import torch
    got = H.sw_batch(ctx, sc, ds, 0, traceback=tb, center_seq=center)
    torch.cuda.synchronize()
    plan, route = ctx.last_plan(), ctx.last_stats()["route"]
    want = H.sw_batch(ctx, sc, ds, 0, traceback=tb, center_seq=center, route=H.HALIGN_ROUTE_INTER)
    torch.cuda.synchronize()
    assert ctx.last_stats()["route"] == 1
    for k in ("score", "cells", "ins", "aligned"):
        if got[k] is not None:
            assert torch.equal(got[k], want[k]), k
    return plan, route


def _center(rng, m):
    import torch
    return torch.from_numpy(rng.integers(0, 20, m).astype(np.uint8)).cuda()


# rows per lane at both ends of the packed kernel's range (2 and 16), around
# its change of wavefronts per SIMD (10, 11), one and two passes; few pairs (one
# per stream, most streams idle) and several per stream; empty sequences
@pytest.mark.parametrize("lanes", [16, 32])
@pytest.mark.parametrize("rows", [2, 10, 11, 12, 16, 17])
@pytest.mark.parametrize("n,streams", [(3, 0), (700, 0), (700, 37)])
def test_packed_score_only(H, ctx, lanes, rows, n, streams, monkeypatch):
    monkeypatch.setenv("HALIGN_STREAM_LANES", str(lanes))
    monkeypatch.setenv("HALIGN_STREAM_PACK", "1")
    if streams:
        monkeypatch.setenv("HALIGN_MAX_STREAMS", str(streams))
    rng = np.random.default_rng(rows * 100 + n)
    seqs = [rng.integers(0, 20, int(L)).astype(np.uint8) for L in rng.integers(1, 90, n)]
    seqs[n // 2] = np.zeros(0, np.uint8)
    seqs[0] = rng.integers(17, 18, 300).astype(np.uint8)
    center = _center(rng, lanes * rows - 3)
    center[5:40] = 17
    ds = H.DeviceSeqs(synth.SeqSet.from_list(seqs))
    for tb in (False, True):
        plan, route = _same(H, ctx, H.Scoring(), ds, center, tb)
        assert plan["packed"] == 1 and route == 0


# batches on both sides of what fills the chip with 64-lane, 32-lane and
# 16-lane streams, and with one center pass and several
@pytest.mark.parametrize("n,lo,hi,m", [(1, 30, 30, 700), (40, 50, 200, 33), (900, 100, 300, 520), (3000, 20, 400, 90),
                                       (9000, 100, 200, 250), (30000, 10, 120, 61)])
def test_default_plan(H, ctx, n, lo, hi, m):
    rng = np.random.default_rng(n)
    ds = H.DeviceSeqs(synth.random_set(rng, n, lo, hi))
    for tb in (False, True):
        _same(H, ctx, H.Scoring(), ds, _center(rng, m), tb)


# 262,144 pairs and more: streams where scores fit, one pair per lane where
# they do not (a matrix entry of 127 on 300 residues)
@pytest.mark.parametrize("tall", [False, True])
def test_default_plan_many_pairs(H, ctx, tall):
    rng = np.random.default_rng(3)
    seqs = synth.random_set(rng, 262144, 0, 24)
    if tall:
        seqs = synth.SeqSet(np.concatenate([seqs.residues, np.full(300, 17, np.uint8)]),
                            np.append(seqs.offsets, len(seqs.residues) + 300))
    mat = synth.BLOSUM62.copy()
    if tall:
        mat[17, 17] = 127
    center = _center(rng, 300 if tall else 20)
    if tall:
        center[:] = 17
    for tb in (False, True):
        plan, route = _same(H, ctx, H.Scoring(mat), H.DeviceSeqs(seqs), center, tb)
        assert route == (1 if tall else 0) and plan["packed"] == (0 if tall else 1)


# batches planned on the device (from 2,048 pairs): the line and its neighbours,
# a last round that is full, empty or nearly so, one pair per stream with empty
# pairs among them, up to 64 rounds and beyond (planned on the host), one and
# several center passes, on each kernel
@pytest.mark.parametrize("lanes,pack", [(64, 0), (32, 0), (16, 0), (32, 1), (16, 1)])
@pytest.mark.parametrize("n,streams,m", [(2047, 0, 70), (2048, 0, 70), (2049, 2048, 40), (2050, 1025, 530),
                                         (2100, 1050, 40), (2100, 33, 40), (2113, 33, 40), (2053, 64, 1100),
                                         (5003, 1000, 300)])
def test_device_plan(H, ctx, n, streams, m, lanes, pack, monkeypatch):
    if lanes != 64:
        monkeypatch.setenv("HALIGN_STREAM_LANES", str(lanes))
    monkeypatch.setenv("HALIGN_STREAM_PACK", str(pack))
    if streams:
        monkeypatch.setenv("HALIGN_MAX_STREAMS", str(streams))
    rng = np.random.default_rng(n + m)
    lens = rng.integers(30, 60, n)
    lens[rng.integers(0, n, 40)] = 0
    lens[rng.integers(0, n, 3)] = 75
    ds = H.DeviceSeqs(synth.SeqSet.from_list([rng.integers(0, 20, int(L)).astype(np.uint8) for L in lens]))
    for tb in (False, True):
        plan, route = _same(H, ctx, H.Scoring(), ds, _center(rng, m), tb)
        assert plan["packed"] == pack and route == 0


# lengths on both sides of the line between the two planners
@pytest.mark.parametrize("lanes,pack", [(64, 0), (32, 1)])
@pytest.mark.parametrize("n,streams,long", [(2048, 700, 60), (3001, 1111, 300), (2500, 65, 8), (4096, 2048, 1)])
def test_device_plan_long_tail(H, ctx, n, streams, long, lanes, pack, monkeypatch):
    if lanes != 64:
        monkeypatch.setenv("HALIGN_STREAM_LANES", str(lanes))
    monkeypatch.setenv("HALIGN_STREAM_PACK", str(pack))
    monkeypatch.setenv("HALIGN_MAX_STREAMS", str(streams))
    rng = np.random.default_rng(n)
    lens = rng.integers(10, 40, n)
    lens[rng.permutation(n)[:long]] = rng.integers(2, 4, long) * 25 * n // streams // 2
    ds = H.DeviceSeqs(synth.SeqSet.from_list([rng.integers(0, 20, int(L)).astype(np.uint8) for L in lens]))
    for tb in (False, True):
        plan, route = _same(H, ctx, H.Scoring(), ds, _center(rng, 90), tb)
        assert plan["packed"] == pack and route == 0


# log-normal lengths: the longest pairs take streams of their own
@pytest.mark.parametrize("lanes,pack", [(64, 0), (16, 1)])
@pytest.mark.parametrize("n,streams", [(4099, 600), (2048, 257), (9000, 3000)])
def test_device_plan_log_normal(H, ctx, n, streams, lanes, pack, monkeypatch):
    if lanes != 64:
        monkeypatch.setenv("HALIGN_STREAM_LANES", str(lanes))
    monkeypatch.setenv("HALIGN_STREAM_PACK", str(pack))
    monkeypatch.setenv("HALIGN_MAX_STREAMS", str(streams))
    rng = np.random.default_rng(n)
    lens = np.clip(40 * np.exp(0.5 * rng.standard_normal(n)), 0, 240).astype(int)
    ds = H.DeviceSeqs(synth.SeqSet.from_list([rng.integers(0, 20, int(L)).astype(np.uint8) for L in lens]))
    for tb in (False, True):
        plan, route = _same(H, ctx, H.Scoring(), ds, _center(rng, 101), tb)
        assert plan["packed"] == pack and route == 0


# whole alignments on the device's plan and on the host's (forced by the dealing
# knob, in chunks under a small workspace, and captured), and with the code
# check's error still raised
@pytest.mark.parametrize("n,center", [(2048, 2047), (6001, 5)])
def test_device_plan_msa(H, ctx, n, center, monkeypatch):
    import torch
    rng = np.random.default_rng(n)
    seqs = synth.random_set(rng, n, 60, 130)
    ds = H.DeviceSeqs(seqs)
    rows = [H.halign_msa(ctx, H.Scoring(), ds, center)[0].cpu().clone()]
    small = H.Context(0, workspace_cap=1 << 20)
    rows.append(H.halign_msa(small, H.Scoring(), ds, center)[0].cpu().clone())
    small.close()
    monkeypatch.setenv("HALIGN_DEAL", "lpt")
    rows.append(H.halign_msa(ctx, H.Scoring(), ds, center)[0].cpu().clone())
    monkeypatch.delenv("HALIGN_DEAL")
    for r in rows[1:]:
        assert torch.equal(r, rows[0])
    bad = ds.residues.clone()
    ds.residues[int(seqs.offsets[n // 2])] = 25
    with pytest.raises(H.HalignError):
        H.halign_msa(ctx, H.Scoring(), ds, center)
    ds.residues.copy_(bad)
    assert torch.equal(H.halign_msa(ctx, H.Scoring(), ds, center)[0].cpu(), rows[0])


# residues staged as aligned words with single bytes at the ends: pairs of 0 .. 9
# residues next to each other at every alignment, codes at and past a small
# alphabet's padding, on both planners; and lengths that the call's first kernel does
# not count
@pytest.mark.parametrize("n", [40, 2300])
def test_staged_residues(H, ctx, n):
    rng = np.random.default_rng(n)
    mat = rng.integers(-4, 6, (5, 5)).astype(np.int8)
    mat = np.minimum(mat, mat.T)
    ds = H.DeviceSeqs(synth.SeqSet.from_list([rng.integers(0, 5, int(L)).astype(np.uint8) for L in rng.integers(0, 10, n)]))
    import torch
    center = torch.from_numpy(rng.integers(0, 5, 37).astype(np.uint8)).cuda()
    for tb in (False, True):
        _same(H, ctx, H.Scoring(mat, 3, 1), ds, center, tb)


@pytest.mark.parametrize("length", [4095, 4096, 9000])
def test_device_plan_long_pairs(H, ctx, length):
    rng = np.random.default_rng(length)
    lens = np.full(2048, length // 2)
    lens[7] = length
    res = rng.integers(0, 20, int(lens.sum())).astype(np.uint8)
    ds = H.DeviceSeqs(synth.SeqSet(res, np.concatenate([[0], np.cumsum(lens)])))
    for tb in (False, True):
        _same(H, ctx, H.Scoring(), ds, _center(rng, 40), tb)
