"""The packed exhaustive center's group tiling (host only; no GPU needed): two
center positions and 64 partners a group, every pair a < b of n positions in exactly
one group and no group idle, and the closed form inverted at block borders up to
the largest sets, where the root of the group number is not exact in a double."""
import numpy as np
import pytest

from test_tiling import H  # noqa: F401  (a fixture)


@pytest.mark.parametrize("n", [0, 1, 2, 3, 4, 63, 64, 65, 66, 127, 128, 129, 191, 200, 257, 300, 449])
def test_every_pair_once(H, n):
    ng = H.halign_exact_tiling(n, H.HALIGN_TILING_PACKED)
    seen = np.zeros((max(n, 1), max(n, 1)), np.int32)
    for g in range(ng):
        _, a, b0 = H.halign_exact_tiling(n, H.HALIGN_TILING_PACKED, g)
        assert a % 2 == 0 and 0 <= a and a + 1 < n and b0 % 64 == 0 and b0 < n   # both centers exist
        b = np.arange(b0, min(b0 + 64, n))
        assert (b > a).any(), (g, a, b0)       # no group is idle
        seen[a, b[b > a]] += 1
        seen[a + 1, b[b > a + 1]] += 1
    assert (seen[np.triu_indices(n, 1)] == 1).all()
    assert seen.sum() == n * (n - 1) // 2


@pytest.mark.parametrize("n", [12345, 10 ** 6, 2 ** 31 - 2, 2 ** 31 - 1])
def test_borders_of_large_sets(H, n):
    nb = (n + 63) // 64
    ng = H.halign_exact_tiling(n, H.HALIGN_TILING_PACKED)
    assert ng == 16 * (nb - 1) * nb + n // 2
    rng = np.random.default_rng(n)
    for q in [0, 1, 2, nb - 3, nb - 2, nb - 1] + [int(x) for x in rng.integers(0, nb, 500)]:
        first, last = 16 * q * (q + 1), min(16 * (q + 1) * (q + 2), ng) - 1   # block q's groups
        for g in (first, first + 1, (first + last) // 2, last):
            assert H.halign_exact_tiling(n, H.HALIGN_TILING_PACKED, g) == (ng, 2 * (g - first), 64 * q)
        assert 2 * (last - first) + 1 == (min(64 * (q + 1), n) - 2 - n % 2 * (q == nb - 1)) + 1


@pytest.mark.parametrize("step", [0, -1, -63, -65, -128])
def test_other_steps_are_refused(H, step):
    with pytest.raises(H.HalignError):
        H.halign_exact_tiling(100, step)
    with pytest.raises(H.HalignError):
        H.halign_exact_tiling(100, H.HALIGN_TILING_PACKED, H.halign_exact_tiling(100, H.HALIGN_TILING_PACKED))
