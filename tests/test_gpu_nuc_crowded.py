"""Nucleotide sets whose segments match by chance more often than anchors fit the
center: the chain's LDS as estimated, outgrown in every sequence (an uneven composition) and
kept larger for the next call, in one sequence of many, and on a set with
more sequences than two a CU; boundary columns and codes that outgrow their
first guess while the lists hold.  Against the oracle, bit for bit."""
import numpy as np
import pytest

from test_gpu_nuc_paths import H, _check, _mutate  # noqa: F401  (H is a fixture)

pytestmark = pytest.mark.gpu


def _draw(rng, n, p):
    return rng.choice(4, n, p=p).astype(np.uint8)


EVEN, UNEVEN = [0.25] * 4, [0.45, 0.05, 0.05, 0.45]


@pytest.mark.parametrize("k,m,p", [(4, 1000, EVEN), (5, 3000, EVEN), (7, 9000, EVEN), (7, 5000, UNEVEN),
                                   (8, 7000, UNEVEN)])
def test_every_sequence(H, k, m, p):
    ctx = H.Context(0)
    rng = np.random.default_rng(k + m)
    c = _draw(rng, m, p)
    seqs = [c] + [_mutate(rng, c, 0.01, 0.001) for _ in range(5)]
    for _ in range(2):   # the second call on what the first one kept
        _check(H, ctx, seqs, k)
    _check(H, ctx, [s[:400] for s in seqs], k)
    _check(H, ctx, seqs, 12)
    ctx.close()


def test_one_of_many(H):
    ctx = H.Context(0)
    rng = np.random.default_rng(3)
    c = _draw(rng, 600, EVEN)
    seqs = [c] + [_mutate(rng, c, 0.01, 0.001) for _ in range(40)] + [np.tile(c, 20)]
    for _ in range(2):
        _check(H, ctx, seqs, 6)
    ctx.close()


def test_more_than_two_a_cu(H):
    ctx = H.Context(0)
    rng = np.random.default_rng(5)
    c = _draw(rng, 400, UNEVEN)
    _check(H, ctx, [c] + [_mutate(rng, c, 0.02, 0.001) for _ in range(700)], 4)
    ctx.close()


# four stretches of 2,500 by 2,500: 1.6 million code words against 270,000
def test_codes_outgrow_their_guess(H):
    rng = np.random.default_rng(6)
    c = _draw(rng, 2600, EVEN)
    for _ in range(2):
        ctx = H.Context(0)
        seqs = [c] + [np.concatenate([c[:50], _draw(rng, 2500, EVEN), c[-50:]]) for _ in range(4)]
        _check(H, ctx, seqs, 16)
        _check(H, ctx, seqs[:2], 16)
        ctx.close()
