"""Level values and statistics at the edges of their pieces: probes per wave
(64), degrees per LDS piece (32), more probes than one round of waves, more
levels than one round of teams; single and batched calls."""
import numpy as np
import pytest

from oracle import cheb, estimator
from paper_2103_10516_amd import workloads as wl

pytestmark = pytest.mark.gpu

CASES = [
    ([31, 32, 33], [63, 64, 65]),
    ([1, 64], [1, 2]),
    ([5], [6300]),  # past 96 waves of 64 probes
    ([2, 40], [3300, 3100]),  # past 48 waves a level
    ([1, 2, 3, 4, 5, 6, 7, 8, 33], [70, 3, 64, 65, 2, 130, 5, 9, 66]),
]


@pytest.mark.parametrize("degrees,m", CASES)
@pytest.mark.parametrize("interp", [False, True])
def test_levels_match_oracle(degrees, m, interp):
    import torch

    from paper_2103_10516_amd import mlct

    g = wl.laplacian_2d(6)
    ctx = mlct.mlct_create(0)
    op = mlct.mlct_op_csr(ctx, *(torch.from_numpy(x).cuda() for x in (g.rowptr, g.col, g.val)))
    mode = mlct.MLCT_DOUBLING | (mlct.MLCT_LEVEL_INTERP if interp else 0)
    r = mlct.mlct_estimate(ctx, op, mlct.MLCT_LOG, 0.01, 8.01, degrees, m, 3, mlct.MLCT_FP64, mode)
    o = estimator.estimate(g.to_scipy(), g.d, cheb.LOG, 0.01, 8.01, degrees, m, 3, doubling=True,
                           level_interp=interp)
    # FP64 throughout: as the estimates' other parity tests (1e-11 relative)
    assert abs(r["value"] - o.value) <= 1e-11 * abs(o.value)
    scale = np.abs(o.level_mean).max()
    np.testing.assert_allclose(r["level_mean"], o.level_mean, rtol=0, atol=1e-11 * scale)
    var = np.array(o.level_var)
    many = np.array(m) > 1
    np.testing.assert_allclose(r["level_var"][many], var[many], rtol=1e-9, atol=1e-20 * g.d)
    item = dict(op=op, kind=mlct.MLCT_LOG, a=0.01, b=8.01, degrees=degrees, m=m, seed=3)
    one = mlct.mlct_estimate(ctx, op, mlct.MLCT_LOG, 0.01, 8.01, degrees, m, 3, mlct.MLCT_FP32,
                             mode)
    two = mlct.mlct_estimate_batch(ctx, [item, dict(item, degrees=[3], m=[65])], mlct.MLCT_FP32,
                                   mode)
    assert two[0]["value"] == one["value"]
    assert np.array_equal(two[0]["level_mean"], one["level_mean"])
    assert np.array_equal(two[0]["level_var"][many], one["level_var"][many])
    ctx.close()
