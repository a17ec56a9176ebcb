"""Which planner a batch takes, by the labels of its host times, with the rows of
every plan equal to the host planner's (which the oracle checks elsewhere):
the device's with and without streams of their own for the longest pairs, and
the host's where the device's rule stops."""
import re

import numpy as np
import pytest

from paper_1704_00878_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import paper_1704_00878_amd as H
    H.lib()
    return H


def _labels(capfd):
    """The labels of the host times printed since the last look, per call."""
    return [re.findall(r" ([a-z_]+) [0-9.]+", line) for line in capfd.readouterr().err.splitlines()
            if line.startswith("halign host us:")]


def _planner(labels):
    return next((x for x in labels if x in ("dplan", "dplan_own", "plan")), None)


def _lens(rng, kind, n):
    if kind == "even":
        return rng.integers(30, 60, n)
    if kind == "log_normal":
        return np.clip(40 * np.exp(0.5 * rng.standard_normal(n)), 0, 240).astype(int)
    lens = rng.integers(10, 40, n)   # few long pairs
    lens[rng.permutation(n)[:20]] = 1200
    return lens


# n, streams, lengths -> the planner, on 64-lane and on packed streams: below the least
# pairs; one round and several; a last round that is nearly full, which the longest
# pairs leave when they take streams of their own; the 64th round and the 65th;
# log-normal lengths; pairs far longer than the average stream (its region would
# be more than four times as long; a stream would be more than 1.3 times the longest pair)
@pytest.mark.parametrize("lanes,pack", [(64, 0), (16, 1)])
@pytest.mark.parametrize("n,streams,kind,want", [
    (2047, 700, "even", "plan"), (2048, 2048, "even", "dplan"), (2048, 700, "even", "dplan_own"), (6001, 1050, "even", "dplan"),
    (2112, 33, "even", "dplan"), (2113, 33, "even", "plan"), (9000, 3000, "log_normal", "dplan_own"),
    (4099, 600, "log_normal", "dplan_own"), (3001, 2000, "few_long", "plan"), (3001, 100, "few_long", "plan")])
def test_planner(H, n, streams, kind, want, lanes, pack, monkeypatch, capfd):
    import torch
    monkeypatch.setenv("HALIGN_HOST_TIMING", "1")
    if lanes != 64:
        monkeypatch.setenv("HALIGN_STREAM_LANES", str(lanes))
    monkeypatch.setenv("HALIGN_STREAM_PACK", str(pack))
    monkeypatch.setenv("HALIGN_MAX_STREAMS", str(streams))
    rng = np.random.default_rng(n + streams)
    seqs = [rng.integers(0, 20, int(L)).astype(np.uint8) for L in _lens(rng, kind, n)]
    seqs[1] = rng.integers(0, 20, 70).astype(np.uint8)
    ds = H.DeviceSeqs(synth.SeqSet.from_list(seqs))
    ctx = H.Context(0)
    _labels(capfd)
    got = H.halign_msa(ctx, H.Scoring(), ds, 1)[0].cpu()
    first = _labels(capfd)
    assert ctx.last_plan()["packed"] == pack
    monkeypatch.setenv("HALIGN_DEAL", "lpt")
    host = H.halign_msa(ctx, H.Scoring(), ds, 1)[0].cpu()
    second = _labels(capfd)
    ctx.close()
    assert torch.equal(got, host)
    assert _planner(second[0]) == "plan"
    assert _planner(first[0]) == want


# a captured batch is planned on the host, and its replays are not planned
def test_captured(H, monkeypatch, capfd):
    import torch
    monkeypatch.setenv("HALIGN_HOST_TIMING", "1")
    rng = np.random.default_rng(2)
    ds = H.DeviceSeqs(synth.random_set(rng, 4000, 60, 130))
    ctx = H.Context(0)
    _labels(capfd)
    want = H.halign_msa(ctx, H.Scoring(), ds, 5)[0].cpu()
    assert _planner(_labels(capfd)[0]) == "dplan"
    ctx.set_graph(True)
    assert torch.equal(H.halign_msa(ctx, H.Scoring(), ds, 5)[0].cpu(), want)
    assert _planner(_labels(capfd)[0]) == "plan"
    for _ in range(3):
        assert torch.equal(H.halign_msa(ctx, H.Scoring(), ds, 5)[0].cpu(), want)
        assert _planner(_labels(capfd)[0]) is None
        out = H.sw_batch(ctx, H.Scoring(), ds, 7)   # an eager batch between the replays, planned on the device
        assert int(out["score"].argmax()) == 7
    assert ctx.graph_launches() == 3
    ctx.close()


# a tuned batch is timed under the planner that then runs it: the device's for all
# candidates but one pair per lane (each is run twice)
@pytest.mark.parametrize("n,want", [(4000, "dplan"), (2000, "plan")])
def test_tuner_times_what_runs(H, n, want, monkeypatch, capfd):
    import torch
    monkeypatch.setenv("HALIGN_HOST_TIMING", "1")
    rng = np.random.default_rng(3)
    ds = H.DeviceSeqs(synth.random_set(rng, n, 100, 130))
    ctx = H.Context(0)
    rows = H.halign_msa(ctx, H.Scoring(), ds, 5)[0].cpu()
    ctx.set_autotune(True)
    _labels(capfd)
    assert torch.equal(H.halign_msa(ctx, H.Scoring(), ds, 5)[0].cpu(), rows)
    first = _labels(capfd)[0]
    assert torch.equal(H.halign_msa(ctx, H.Scoring(), ds, 5)[0].cpu(), rows)
    again = _labels(capfd)[0]
    ctx.close()
    trials = first[:first.index("tune")]
    assert "tune" in again and _planner(again[:again.index("tune")]) is None
    if "p_deal" in again or _planner(again) != "plan":   # streams were chosen
        assert _planner(again) == want
    assert trials.count(want) >= 2 * 6
    assert trials.count("plan") + trials.count("dplan") + trials.count("dplan_own") >= 2 * 7

