"""The column profile and the SP scores at the sizes where their launches
change, against the oracle (integers, compared exactly): widths around a
lane's four columns and a workgroup's 256, row counts around a wavefront's
batches and a slab, an MSA at every byte alignment, many calls on kept
scratch, and two threads at once."""
import threading

import numpy as np
import pytest

import oracle
from paper_1704_00878_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import paper_1704_00878_amd as H
    return H


def _msa(rng, n, w, alpha=24, gap=0.3):
    a = rng.integers(0, alpha, (n, w)).astype(np.uint8)
    a[rng.random((n, w)) < gap] = 255
    return a


def _check(H, a, dev):
    from oracle_par import sp_from_profile
    want = oracle.column_profile(a, 24)
    assert (H.halign_column_profile(dev).cpu().numpy() == want).all()
    assert H.halign_sp_score(H.Scoring(), dev) == sp_from_profile(want, np.asarray(synth.BLOSUM62, np.int8), 1)


@pytest.mark.parametrize("n,w", [(1, 1), (3, 2), (9, 3), (65, 4), (127, 5), (129, 255), (257, 257), (1, 4097),
                                 (70, 4500)])
def test_shapes(H, n, w):
    import torch
    ctx = H.Context(0)   # scratch is kept while a context lives
    a = _msa(np.random.default_rng(n + 1000 * w), n, w)
    buf = torch.zeros(n * w + 8, dtype=torch.uint8, device="cuda")
    for off in range(4):
        dev = buf[off:off + n * w].view(n, w)
        dev.copy_(torch.from_numpy(a))
        _check(H, a, dev)
    bad = a.copy()
    bad[n - 1, w - 1] = 77
    with pytest.raises(H.HalignError):
        H.halign_column_profile(torch.from_numpy(bad).cuda())
    with pytest.raises(H.HalignError):
        H.halign_sp_score(H.Scoring(), torch.from_numpy(bad).cuda())
    _check(H, a, torch.from_numpy(a).cuda())   # the flag of a failed call does not outlive it
    ctx.close()
    _check(H, a, torch.from_numpy(a).cuda())   # and without one


def test_two_threads(H):
    import torch
    ctx = H.Context(0)
    sets = [_msa(np.random.default_rng(k), 200 + 300 * k, 300 + 77 * k) for k in range(2)]
    errs = []

    def work(a):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                dev = torch.from_numpy(a).cuda()
                for _ in range(20):
                    _check(H, a, dev)
        except Exception as e:
            errs.append(e)

    ths = [threading.Thread(target=work, args=(a,)) for a in sets]
    for t in ths:
        t.start()
    for t in ths:
        t.join()
    assert not errs, errs
    ctx.close()
