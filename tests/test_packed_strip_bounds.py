"""The packed strip kernel's arithmetic on the host (no GPU needed): strips of 32
rows whose row pairs hold every value plus a multiple of the gap extension, with
the maxima as halves, against the oracle at scores and gap costs up to the
bounds of the host's rule, every operand checked to stay in range."""
import os
import re

import numpy as np
import pytest

import oracle
from test_packed_bounds import CSRC, _constants

ROWS = 32


def _rule():
    host = open(os.path.join(CSRC, "halign.hip")).read()
    m = re.search(r"return S\.goe <= 256 && S\.ge <= 256 && top < (\d+) && top \+ (\d+) \* S\.ge < (\d+);", host)
    return [int(x) for x in m.groups()]


def _sw_strips(S, go, ge, c, s, B, P):
    """The best H as the kernel computes it, one center and one partner."""
    def half(v):    # an operand of a half maximum
        assert 0 <= v < 0x7C00, v
        return v

    def short(v):   # an operand of an integer maximum, or any other value held
        assert -0x8000 <= v < 0x8000, v
        return v

    goe, n = go + ge, len(s)
    flo = [B + ge * (k + 2) for k in range(ROWS // 2)]
    hm = [f - ge for f in flo]
    bound = [(B - go, B - go)] * n          # hg and F* above the strip, per column
    for i0 in range(0, len(c), ROWS):
        hg = [flo[t // 2] - ge - go for t in range(ROWS)]
        e = list(hg)
        diag0 = B - go
        for j in range(n):
            upg, upf = bound[j]
            diag, diag0 = diag0, upg
            for t in range(ROWS):
                k = t // 2
                real = i0 + t < len(c)
                p = int(S[c[i0 + t], s[j]]) + (go if t & 1 else goe) if real else P
                en = short(max(half(e[t]), half(hg[t]), half(flo[k])) - ge)
                fn = short(max(short(upf), short(upg)) - (ge if t & 1 else 0))
                h = max(half(diag + p), half(en), half(fn))
                assert real or diag + p < en        # a padding entry is never a source
                hm[k] = max(half(hm[k]), h)
                diag, hg[t], e[t] = hg[t], short(h - go), en
                upg, upf = hg[t], fn
            bound[j] = (short(upg - ROWS // 2 * ge), short(upf - ROWS // 2 * ge))
    return max(hm[k] - (flo[k] - ge) for k in range(ROWS // 2))


# a diagonal of 50: 298 residues score 14,900, which go + ge and 18 ge take to the
# rule's bounds; gap costs at their ends; one strip, ragged ones and several
@pytest.mark.parametrize("go,ge,m,n", [
    (44, 55, 298, 298), (98, 1, 298, 298), (0, 55, 298, 298), (11, 1, 299, 299), (44, 55, 298, 150), (0, 1, 33, 90),
    (200, 56, 200, 200), (0, 256, 65, 80), (255, 1, 64, 64), (3, 2, 1, 40), (11, 1, 95, 1)])
def test_strips_match_the_oracle_up_to_the_bounds(go, ge, m, n):
    B, P, _ = _constants()
    low, offsets, high = _rule()
    assert ROWS // 2 + 2 == offsets     # the last row pair's floor, one ge above its values
    rng = np.random.default_rng(m + go)
    S = rng.integers(-128, 10, size=(4, 4)).astype(np.int8)
    np.fill_diagonal(S, [50, 7, 3, 1])
    top = 50 * max(m, n) + go + ge
    assert top < low and top + offsets * ge < high
    for kind in ("same", "near", "any"):
        if kind == "any":
            c, s = rng.integers(0, 4, m).astype(np.uint8), rng.integers(0, 4, n).astype(np.uint8)
        else:
            c, s = np.zeros(m, np.uint8), np.zeros(n, np.uint8)
            if kind == "near":
                c[rng.random(m) < 0.05] = 1
                s[rng.random(n) < 0.05] = 2
        got, ref = _sw_strips(S, go, ge, c, s, B, P), oracle.sw(S, go, ge, c, s)["score"]
        assert got == ref, (kind, got, ref)
        if kind == "same":
            assert got == 50 * min(m, n)
