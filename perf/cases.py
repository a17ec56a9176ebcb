"""The calls whose time counts in this library, as cases that can be prepared and run.

Each case is one pass through the public entry points on inputs that a seed
makes: the protein MSA from a handful of sequences to hundreds of thousands
(the one-pair-per-lane range), a score-only search, the exact center, the
learned center's proposer and its training step, the nucleotide MSA, the tree,
the distances and the SP evaluation.  Sizes follow the sets of synth.py,
bench.py and the tests; `draw` spreads them over the ranges between.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1704_00878_amd as H
from paper_1704_00878_amd import synth

DEV = "cuda:0"


def listed():
    return [
        # a handful of short proteins aligned interactively: latency and launches
        {"name": "msa_64", "kind": "msa", "n": 64, "lo": 80, "hi": 160, "m": 120, "roots": 1, "p_sub": 0.20,
         "p_indel": 0.05, "tuned": False},
        # the benchmark's batch: 20,000 domain-length proteins, plans tuned once per context as bench.py does
        {"name": "msa_batch20k", "kind": "msa", "n": 20000, "lo": 200, "hi": 500, "m": 311, "roots": 8, "p_sub": 0.25,
         "p_indel": 0.05, "tuned": True},
        # a long-tailed protein family against a short center, plans left at their defaults
        {"name": "msa_longtail", "kind": "msa", "n": 50001, "lo": 50, "hi": 2000, "m": 101, "roots": 32, "p_sub": 0.30,
         "p_indel": 0.08, "tuned": False},
        # a whole database's worth of sequences: one pair per lane, gigabytes of codes and rows
        {"name": "msa_300k", "kind": "msa", "n": 300000, "lo": 50, "hi": 1000, "m": 200, "roots": 128, "p_sub": 0.30,
         "p_indel": 0.06, "tuned": False},
        # a query scored against a set (no traceback): end cells and scores only
        {"name": "search_20k", "kind": "search", "n": 20011, "lo": 150, "hi": 600, "m": 400, "roots": 32,
         "p_sub": 0.25, "p_indel": 0.05},
        # the exact center of a mid-sized family: all pairs, scores only
        {"name": "center_exact_1500", "kind": "exact", "n": 1500, "lo": 150, "hi": 600, "roots": 8, "p_sub": 0.25,
         "p_indel": 0.05},
        # the proposer over a set: features, embedding, candidate scores, top candidates
        {"name": "propose_16k", "kind": "propose", "n": 16384, "lo": 150, "hi": 600, "k": 16},
        # one training step of the proposer: forward, loss, backward, Adam on every tensor
        {"name": "train_step_1024", "kind": "train", "pairs": 1024, "lo": 150, "hi": 600},
        # hundreds of mitochondrial genomes: anchors, stretches, merge, rows
        {"name": "nuc_672", "kind": "nuc", "n": 672, "length": 16569, "p_sub": 0.003, "p_indel": 0.0002, "k": 16},
        # the tree of such an alignment: distances, clustering, neighbour joining
        {"name": "tree_672", "kind": "tree", "n": 672, "w": 18611, "p_sub": 0.003, "p_gap": 0.11},
        # all p-distances of a protein alignment
        {"name": "pdist_3001", "kind": "pdist", "n": 3001, "w": 4030, "p_sub": 0.25, "p_gap": 0.9},
        # the evaluation of a protein alignment: both SP scores and its column profile
        {"name": "sp_20k", "kind": "sp", "n": 20000, "w": 4030, "p_sub": 0.25, "p_gap": 0.9},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["msa", "msa", "msa", "search", "exact", "propose", "train", "nuc", "tree", "pdist", "sp"])
    lo = rng.randint(50, 200)
    hi = lo + rng.randint(60, 500)
    fam = {"lo": lo, "hi": hi, "roots": rng.randint(1, 64), "p_sub": round(rng.uniform(0.1, 0.35), 3),
           "p_indel": round(rng.uniform(0.02, 0.08), 3)}
    if kind == "msa":
        n = _log(rng, 3, 300000)
        top = 300000 * 525.0 * 200.0 / (n * (lo + hi) / 2.0)   # center length at the largest listed case's cells
        return {"kind": "msa", "n": n, "m": int(min(rng.randint(lo, hi), max(lo, top))), **fam,
                "tuned": rng.random() < 0.25}
    if kind == "search":
        return {"kind": "search", "n": _log(rng, 1, 20011), "m": rng.randint(lo, min(hi, 400)), **fam}
    if kind == "exact":
        return {"kind": "exact", "n": _log(rng, 8, 1400), **{**fam, "hi": min(hi, 500)}}
    if kind == "propose":
        return {"kind": "propose", "n": _log(rng, 20, 16384), "lo": lo, "hi": min(hi, 550),
                "k": rng.choice([1, 5, 16, 16, 64])}
    if kind == "train":
        return {"kind": "train", "pairs": _log(rng, 16, 1024), "lo": lo, "hi": hi}
    if kind == "nuc":
        return {"kind": "nuc", "n": _log(rng, 8, 640), "length": _log(rng, 700, 16000),
                "p_sub": round(rng.uniform(0.001, 0.004), 4), "p_indel": round(rng.uniform(0.0001, 0.0003), 5),
                "k": rng.choice([12, 16, 16, 24])}
    if kind == "tree":
        return {"kind": "tree", "n": _log(rng, 24, 640), "w": _log(rng, 600, 18000),
                "p_sub": round(rng.uniform(0.003, 0.03), 4), "p_gap": round(rng.uniform(0.02, 0.2), 3)}
    if kind == "pdist":
        return {"kind": "pdist", "n": _log(rng, 30, 3000), "w": _log(rng, 120, 4000),
                "p_sub": round(rng.uniform(0.05, 0.3), 3), "p_gap": round(rng.uniform(0.1, 0.9), 3)}
    return {"kind": "sp", "n": _log(rng, 60, 20000), "w": _log(rng, 120, 4000),
            "p_sub": round(rng.uniform(0.05, 0.3), 3), "p_gap": round(rng.uniform(0.1, 0.9), 3)}


# ---------------------------------------------------------------------------
# Inputs (made on the GPU from the seed)
# ---------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(DEV)
    g.manual_seed(20170403 + int(seed))
    return g


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device=DEV)


def _background(g, k):
    cdf = torch.tensor(np.cumsum(synth.BACKGROUND)[:-1], dtype=torch.float32, device=DEV)
    return torch.searchsorted(cdf, _rand(g, k), right=True).to(torch.uint8)


def _mutate(g, base, ends, p_sub, p_indel, letters, inserted):
    """Substitutions and indels of concatenated sequences that end at `ends`."""
    T = base.numel()
    hit = _rand(g, T) < p_sub
    other = torch.randint(1, letters, (T,), generator=g, device=DEV, dtype=torch.uint8)
    base = torch.where(hit, (base + other) % letters, base)
    u = _rand(g, T)
    keep = u >= p_indel                                    # one residue in every p_indel is lost
    grow = (u > 1.0 - 0.5 * p_indel) & keep                # insertions, geometric(0.5) residues
    length = torch.floor(torch.log2(1.0 / (1.0 - _rand(g, T)).clamp_min(1e-6))).to(torch.int64) + 1
    out_end = torch.cumsum(keep.to(torch.int64) + torch.where(grow, length, 0), 0)
    out = inserted(int(out_end[-1]))
    out[out_end[keep] - 1] = base[keep]
    off = torch.zeros(ends.numel() + 1, dtype=torch.int64, device=DEV)
    off[1:] = out_end[ends - 1]
    return synth.SeqSet(out.cpu().numpy(), off.cpu().numpy())


def _proteins(g, n, lo, hi, roots, p_sub, p_indel):
    """n relatives of a few random roots (windows of a root, padded where the
    root is shorter), substituted and with indels; hi >= 2000: a long tail."""
    def law(k):
        if hi >= 2000:
            z = torch.randn(k, generator=g, device=DEV)
            return torch.exp(5.8 + 0.5 * z).round().clamp(lo, hi).to(torch.int64)
        return torch.randint(lo, hi + 1, (k,), generator=g, device=DEV)
    rl = law(roots)
    ro = torch.zeros(roots + 1, dtype=torch.int64, device=DEV)
    ro[1:] = torch.cumsum(rl, 0)
    table = _background(g, int(ro[-1]))
    which = torch.randint(0, roots, (n,), generator=g, device=DEV)
    L = law(n)
    take = torch.minimum(L, rl[which])
    start = (_rand(g, n) * (rl[which] - take + 1)).to(torch.int64)
    left = (_rand(g, n) * (L - take + 1)).to(torch.int64)
    ends = torch.cumsum(L, 0)
    k = torch.repeat_interleave(torch.arange(n, device=DEV), L)
    q = torch.arange(int(ends[-1]), device=DEV) - (ends - L)[k] - left[k]
    inside = (q >= 0) & (q < take[k])
    at = (ro[which] + start)[k] + q
    base = torch.where(inside, table[at.clamp(0, table.numel() - 1)], _background(g, q.numel()))
    del k, q, inside, at
    return _mutate(g, base, ends, p_sub, p_indel, 20, lambda t: _background(g, t))


def _genomes(g, n, length, p_sub, p_indel):
    root = torch.randint(0, 4, (length,), generator=g, device=DEV, dtype=torch.uint8)
    ends = torch.arange(1, n + 1, device=DEV) * length
    return _mutate(g, root.repeat(n), ends, p_sub, p_indel, 4,
                   lambda t: torch.randint(0, 4, (t,), generator=g, device=DEV, dtype=torch.uint8))


def _alignment(g, n, w, letters, p_sub, p_gap, families):
    """An n x w alignment: columns that every row holds and, a share p_gap,
    columns that only few rows hold."""
    roots = torch.randint(0, letters, (families, w), generator=g, device=DEV, dtype=torch.uint8)
    msa = roots[torch.randint(0, families, (n,), generator=g, device=DEV)]
    hit = _rand(g, n, w) < p_sub
    other = torch.randint(1, letters, (n, w), generator=g, device=DEV, dtype=torch.uint8)
    msa = torch.where(hit, (msa + other) % letters, msa)
    rare = _rand(g, w) < p_gap
    gone = _rand(g, n, w) < torch.where(rare, 0.98, 0.01)[None, :]
    return msa.masked_fill_(gone, H.GAP)


def _features(seqs):
    """3-mer counts of every sequence (fp32)."""
    n = seqs.n
    r = torch.from_numpy(seqs.residues).to(DEV).to(torch.int64)
    off = torch.from_numpy(seqs.offsets).to(DEV)
    row = torch.repeat_interleave(torch.arange(n, device=DEV), off[1:] - off[:-1])
    a, b, c = r[:-2], r[1:-1], r[2:]
    ok = (row[:-2] == row[2:]) & (a < 20) & (b < 20) & (c < 20)
    at = row[:-2] * H.FEAT + 400 * a + 20 * b + c
    return torch.bincount(at[ok], minlength=n * H.FEAT).view(n, H.FEAT).float()


def _sequences(case, seed):
    return _proteins(_gen(seed), case["n"], case["lo"], case["hi"], case.get("roots", 32), case.get("p_sub", 0.25),
                     case.get("p_indel", 0.05))


def _params(g):
    l1, l2 = math.sqrt(6.0 / H.FEAT), math.sqrt(6.0 / H.HID)
    return [(_rand(g, H.FEAT, H.HID) * 2 - 1) * l1, (_rand(g, H.HID) - 0.5) * 0.1,
            (_rand(g, H.HID, H.EMB) * 2 - 1) * l2, (_rand(g, H.EMB) - 0.5) * 0.1]


def _train_inputs(case, seed):
    g = _gen(seed)
    P = case["pairs"]
    X = _features(_proteins(g, 2 * P, case["lo"], case["hi"], 32, 0.25, 0.05)).to(torch.bfloat16)
    params = _params(g)
    target = 0.3 + 4.0 * _rand(g, P) * _rand(g, P)
    moments = [(torch.randn(p.shape, generator=g, device=DEV) * 1e-3,
                (_rand(g, *p.shape) + 0.5) * 1e-5) for p in params]
    return X, params, target, moments


LR, B1, B2, EPS, STEP = 1e-3, 0.9, 0.999, 1e-8, 200


def prepare(case, seed):
    kind = case["kind"]
    g = _gen(seed)
    if kind in ("msa", "search", "exact", "propose", "nuc"):
        seqs = _genomes(g, case["n"], case["length"], case["p_sub"], case["p_indel"]) if kind == "nuc" \
            else _sequences(case, seed)
        s = {"kind": kind, "ctx": H.Context(0), "ds": H.DeviceSeqs(seqs, DEV), "sc": H.Scoring()}
        if kind in ("msa", "search"):   # the center: the first sequence whose length is nearest m
            s["center"] = int(np.argmin(np.abs(seqs.lengths() - case["m"])))
        if kind == "msa":
            s["ctx"].set_autotune(case["tuned"])
            # the buffer a program keeps for the rows; the width is known only after the merge
            s["out"] = torch.zeros(case["n"] * int(2.4 * case["hi"] + 24 * case["m"] + 300), dtype=torch.uint8, device=DEV)
        if kind == "nuc":
            s["out"] = torch.zeros(case["n"] * int(1.5 * case["length"] + 500), dtype=torch.uint8, device=DEV)
            s["sc"] = H.Scoring(synth.NUC_MATRIX, synth.NUC_GAP_OPEN, synth.NUC_GAP_EXTEND)
            s["k"] = case["k"]
        if kind == "propose":
            p = H.Proposer(params=[x.cpu().numpy() for x in _params(_gen(seed + 1000003))], device=DEV)
            s.update(prop=p, k=min(case["k"], case["n"]))
        return s
    if kind == "train":
        X, params, target, moments = _train_inputs(case, seed)
        P = case["pairs"]
        f = dict(dtype=torch.float32, device=DEV)
        return {"kind": kind, "ctx": H.Context(0), "P": P, "X": X.view(torch.int16), "target": target, "t": STEP,
                "prop": H.Proposer(params=[x.cpu().numpy() for x in params], device=DEV), "moments": moments,
                "Z": torch.empty(2 * P, H.HID, **f), "E": torch.empty(2 * P, H.EMB, **f),
                "Hb": torch.empty(2 * P, H.HID, dtype=torch.int16, device=DEV),
                "dE": torch.empty(2 * P, H.EMB, **f), "loss": torch.empty(1, **f),
                "grads": [torch.empty(H.FEAT, H.HID, **f), torch.empty(H.HID, **f),
                          torch.empty(H.HID, H.EMB, **f), torch.empty(H.EMB, **f)]}
    n, w = case["n"], case["w"]
    if kind == "tree":
        return {"kind": kind, "ctx": H.Context(0), "msa": _alignment(g, n, w, 4, case["p_sub"], case["p_gap"], 1),
                "perm": synth.tree_permutation(n, seed=seed)}
    msa = _alignment(g, n, w, 20, case["p_sub"], case["p_gap"], 8)
    return {"kind": kind, "ctx": H.Context(0), "msa": msa, "sc": H.Scoring()}


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def _rows(s, msa):
    """The row buffer whole, or the alignment itself where it did not fit."""
    return s["out"] if msa.data_ptr() == s["out"].data_ptr() else msa


def run(s):
    kind = s["kind"]
    if kind == "msa":
        msa, c = H.halign_msa(s["ctx"], s["sc"], s["ds"], s["center"], out=s["out"])
        return {"msa": _rows(s, msa), "width": msa.shape[1], "center": c}
    if kind == "search":
        out = H.sw_batch(s["ctx"], s["sc"], s["ds"], s["center"], traceback=False)
        return {"score": out["score"], "cells": out["cells"]}
    if kind == "exact":
        sums = torch.empty(s["ds"].n, dtype=torch.int64, device=DEV)
        c = H.halign_center_exact(s["ctx"], s["sc"], s["ds"], sums)
        return {"sums": sums, "center": c}
    if kind == "propose":
        n = s["ds"].n
        X = torch.empty(n, H.FEAT, dtype=torch.int16, device=DEV)
        H.halign_featurize(s["ds"], X)
        Hb = torch.empty(n, H.HID, dtype=torch.int16, device=DEV)
        E = torch.empty(n, H.EMB, dtype=torch.float32, device=DEV)
        H.halign_mlp_forward(s["ctx"], s["prop"], X, n, None, Hb, E)
        u = torch.empty(n, dtype=torch.float32, device=DEV)
        top = torch.empty(s["k"], dtype=torch.int32, device=DEV)
        H.halign_topk_center(s["ctx"], E, n, s["k"], u, top)
        return {"X": X.view(torch.bfloat16), "Hb": Hb.view(torch.bfloat16), "E": E, "u": u, "top": top}
    if kind == "train":
        ctx, prop, P = s["ctx"], s["prop"], s["P"]
        H.halign_mlp_forward(ctx, prop, s["X"], 2 * P, s["Z"], s["Hb"], s["E"])
        H.halign_pair_loss(ctx, s["E"], s["target"], P, s["dE"], s["loss"])
        H.halign_mlp_backward(ctx, prop, s["X"], 2 * P, s["Z"], s["Hb"], s["dE"], *s["grads"])
        s["t"] += 1
        tensors = [(prop.W1, prop.W1b), (prop.b1, None), (prop.W2, prop.W2b), (prop.b2, None)]
        for (p, pb), d, (m, v) in zip(tensors, s["grads"], s["moments"]):
            H.halign_adam_step(p, d, m, v, pb, LR, B1, B2, EPS, s["t"])
        return {"E": s["E"], "loss": s["loss"], "dE": s["dE"], "grads": s["grads"], "moments": s["moments"],
                "weights": [p for p, _ in tensors], "copies": [b.view(torch.bfloat16) for _, b in tensors if b is not None]}
    if kind == "nuc":
        msa, score = H.halign_nuc_msa(s["ctx"], s["sc"], s["ds"], s["k"], out=s["out"])
        return {"msa": _rows(s, msa), "width": msa.shape[1], "score": score}
    if kind == "tree":
        parent, blen = H.halign_nj_tree(s["ctx"], s["msa"], s["perm"])
        pad = (0, 2 * s["msa"].shape[0] + 2 - len(parent))   # the node count depends on the clusters
        return {"parent": np.pad(parent, pad), "blen": np.pad(blen, pad), "nodes": len(parent)}
    if kind == "pdist":
        return H.halign_pdist(s["ctx"], s["msa"])
    sp, bl = H.halign_sp_score(s["sc"], s["msa"])
    return {"sp": sp, "blosum": bl, "profile": H.halign_column_profile(s["msa"])}


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    kind = case["kind"]
    n = case.get("n", 0)
    mean = 350.0 if case.get("hi", 0) >= 2000 else (case.get("lo", 0) + case.get("hi", 0)) / 2.0
    if kind == "msa":   # 14 integer operations per cell with traceback; rows about 12 columns per center residue
        m = case["m"]
        return {"bytes": n * (mean + 12.0 * m), "flops": 14.0 * n * mean * m}
    if kind == "search":
        return {"bytes": n * (mean + 20.0), "flops": 9.0 * n * mean * case["m"]}
    if kind == "exact":
        return {"bytes": n * mean, "flops": 9.0 * n * (n - 1) / 2 * mean * mean}
    if kind == "propose":   # features, activations, embedding and scores written once
        return {"bytes": n * (mean + 2.0 * H.FEAT + 2.0 * H.HID + 4.0 * H.EMB + 4.0) + 2.0 * H.FEAT * H.HID,
                "flops": 2.0 * n * (H.FEAT * H.HID + H.HID * H.EMB)}
    if kind == "train":   # features read once; p, m, v read and written, the bf16 copy and the gradient written
        r = 2.0 * case["pairs"]
        par = H.FEAT * H.HID + H.HID * H.EMB
        return {"bytes": r * (2.0 * H.FEAT + 6.0 * H.HID + 8.0 * H.EMB) + par * (24.0 + 4.0 + 4.0),
                "flops": 2.0 * r * (2.0 * H.FEAT * H.HID + 3.0 * H.HID * H.EMB)}
    if kind == "nuc":
        return {"bytes": n * case["length"] * 2.1, "flops": 4.0 * n * case["length"]}
    w = case["w"]
    if kind == "tree":   # sample and cluster distances, and the joins of the clusters' seeds
        k = n / 2.0
        return {"bytes": 1.0 * n * w, "flops": 0.75 * w * (0.1 * n * n + k * k / 2) + k ** 3}
    if kind == "pdist":
        return {"bytes": n * w + 8.0 * n * n, "flops": 0.75 * w * n * n / 2}
    return {"bytes": 1.0 * n * w + 100.0 * w, "flops": 1.0 * n * w}


# ---------------------------------------------------------------------------
# The computed numbers in 64 bits
# ---------------------------------------------------------------------------
def _embed64(X, params):
    W1, b1, W2, b2 = [p.double() for p in params]
    Z = X.double() @ W1.to(torch.bfloat16).double() + b1
    A = Z.clamp_min(0.0)
    return Z, A, A @ W2.to(torch.bfloat16).double() + b2


def exact(case, seed):
    kind = case["kind"]
    if kind == "propose":
        X = _features(_sequences(case, seed))
        params = _params(_gen(seed + 1000003))
        parts = [_embed64(x, params)[1:] for x in X.split(4096)]
        A, E = torch.cat([p[0] for p in parts]), torch.cat([p[1] for p in parts])
        u = (E * (E.sum(0) - E)).sum(1)
        return {"X": X, "Hb": A, "E": E, "u": u, "top": None}
    if kind == "train":
        X, params, target, moments = _train_inputs(case, seed)
        P = case["pairs"]
        X = X.double()
        Z, A, E = _embed64(X, params)
        W2 = params[2].to(torch.bfloat16).double()
        diff = (E[:P] * E[P:]).sum(1) - target.double()
        scale = (2.0 * diff / P)[:, None]
        dE = torch.cat([scale * E[P:], scale * E[:P]])
        dZ = (dE @ W2.t()) * (Z > 0)
        grads = [X.t() @ dZ, dZ.sum(0), A.t() @ dE, dE.sum(0)]
        t, weights, new = STEP + 1, [], []
        for p, d, (m, v) in zip(params, grads, moments):
            m = B1 * m.double() + (1 - B1) * d
            v = B2 * v.double() + (1 - B2) * d * d
            new.append((m, v))
            weights.append(p.double() - LR * (m / (1 - B1 ** t)) / ((v / (1 - B2 ** t)).sqrt() + EPS))
        return {"E": E, "loss": (diff * diff).mean().reshape(1), "dE": dE, "grads": grads, "moments": new,
                "weights": weights, "copies": [weights[0], weights[2]]}
    if kind == "pdist":
        msa = _alignment(_gen(seed), case["n"], case["w"], 20, case["p_sub"], case["p_gap"], 8)
        held = (msa != H.GAP).float()
        both = (held @ held.t()).double()   # counts below 2^24: exact in fp32
        same = torch.zeros_like(both)
        for a in range(20):
            h = (msa == a).float()
            same += (h @ h.t()).double()
        return torch.where(both > 0, (both - same) / both.clamp_min(1.0), 1.0)
    return None
