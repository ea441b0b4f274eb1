"""Operators without entries (A = 0, no column array): one probe block, and the
block counts that run in shared launches, as a single estimate and in batches of
both launch forms, against the FP64 oracle."""
import numpy as np
import pytest
import scipy.sparse as sp

from oracle import cheb, estimator

pytestmark = pytest.mark.gpu

D = 1000
A0, B0 = -1.0, 2.0
LEVELS = {1: ([9], [40]), 3: ([4, 9], [70, 20]), 4: ([2, 4, 9], [70, 64, 5])}


@pytest.mark.parametrize("pattern", [False, True])
@pytest.mark.parametrize("blocks", sorted(LEVELS))
def test_no_entries(blocks, pattern):
    import torch

    from paper_2103_10516_amd import mlct

    degrees, m = LEVELS[blocks]
    assert sum(-(-k // 64) for k in m) == blocks
    ctx = mlct.mlct_create(0)
    col = torch.empty(0, dtype=torch.int32, device="cuda")
    val = None if pattern else torch.empty(0, dtype=torch.float32, device="cuda")
    op = mlct.mlct_op_csr(ctx, torch.zeros(D + 1, dtype=torch.int32, device="cuda"), col, val)
    for mode, doubling in ((mlct.MLCT_DIRECT, False), (mlct.MLCT_DOUBLING, True)):
        o = estimator.estimate(sp.csr_matrix((D, D)), D, cheb.EXP, A0, B0, degrees, m, 3,
                               doubling=doubling)
        # V_k = T_k(beta) z with |beta| < 1: n steps of rounding at most
        tol = 10 * degrees[-1] ** 2 * 2.0**-24 * D * np.exp(B0)
        item = dict(op=op, kind=mlct.MLCT_EXP, a=A0, b=B0, degrees=degrees, m=m, seed=3)
        got = [mlct.mlct_estimate(ctx, op, mlct.MLCT_EXP, A0, B0, degrees, m, 3, mlct.MLCT_FP32,
                                  mode)]
        for form in (mlct.MLCT_BATCH_LOCKSTEP, mlct.MLCT_BATCH_PERSISTENT):
            got += mlct.mlct_estimate_batch(ctx, [item, dict(item, seed=3)], mlct.MLCT_FP32,
                                            mode | form)
        assert abs(got[0]["value"] - o.value) <= tol
        for r in got[1:]:
            assert r["value"] == got[0]["value"]
    op.close()
    ctx.close()
