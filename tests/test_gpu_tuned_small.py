"""First tuned calls of fresh contexts on small batches, whose trials follow the
matrix's copy closely: the same results as untuned ones, which the oracle checks
elsewhere."""
import numpy as np
import pytest

from paper_1704_00878_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tb", [True, False])
@pytest.mark.parametrize("n", [1, 2, 5, 64, 300, 1500, 2000])
def test_first_tuned_call(n, tb):
    import torch
    import paper_1704_00878_amd as H
    rng = np.random.default_rng(n)
    ds = H.DeviceSeqs(synth.random_set(rng, n, 100, 130))
    ctx = H.Context(0)
    want = H.sw_batch(ctx, H.Scoring(), ds, 0, traceback=tb)
    torch.cuda.synchronize()
    ctx.close()
    for _ in range(8):
        ctx = H.Context(0)
        H.sw_batch(ctx, H.Scoring(), ds, 0, traceback=tb)   # the buffers are there, the plan is not
        ctx.set_autotune(True)
        got = H.sw_batch(ctx, H.Scoring(), ds, 0, traceback=tb)
        torch.cuda.synchronize()
        ctx.close()
        for k, w in want.items():
            assert got[k] is None or k == "m" or torch.equal(got[k], w), k
