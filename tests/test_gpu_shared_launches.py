"""Estimates that run their probe blocks in shared launches against the same
estimates block by block (the batch's solo threshold below the operator's rows),
bit for bit; which of the two a call takes; and the errors of either."""
import numpy as np
import pytest

from paper_2103_10516_amd import workloads as wl
from tests.test_gpu_long_rows import _matrix, ctx  # noqa: F401

pytestmark = pytest.mark.gpu


def _op(ctx, g):  # noqa: F811
    import torch

    from paper_2103_10516_amd import mlct

    return mlct.mlct_op_csr(ctx, *(None if x is None else torch.from_numpy(x).cuda()
                                   for x in (g.rowptr, g.col, g.val)))


def _estimate(ctx, op, *args, alone=False):  # noqa: F811
    """The estimate and whether it ran in shared launches."""
    from paper_2103_10516_amd import mlct

    mlct.mlct_set_option(ctx, mlct.MLCT_OPT_BATCH_SOLO_ROWS, 1 if alone else 0)
    mlct.mlct_timing(ctx, True)
    try:
        r = mlct.mlct_estimate(ctx, op, *args)
    finally:
        mlct.mlct_timing(ctx, False)
        mlct.mlct_set_option(ctx, mlct.MLCT_OPT_BATCH_SOLO_ROWS, 0)
    shared, single = (mlct.mlct_timing_read(ctx, k)[0] > 0
                      for k in (mlct.MLCT_KERNEL_BATCH_STEP, mlct.MLCT_KERNEL_CSR_STEP))
    assert shared != single
    return r, shared


def _same(x, y):
    assert x["value"] == y["value"] and x["est_var"] == y["est_var"]
    assert x["max_moment_ratio"] == y["max_moment_ratio"]
    np.testing.assert_array_equal(x["level_mean"], y["level_mean"])
    np.testing.assert_array_equal(x["level_var"], y["level_var"])


# degrees, probes, and whether shared launches save enough steps (symmetric form)
LEVELS = [([10, 30], [70, 20], True), ([6, 12, 24], [64, 5, 2], True), ([24], [192], True),
          ([10, 20], [64, 64], False), ([2, 40], [65, 64], False), ([2, 4], [65, 2], False)]


@pytest.mark.parametrize("form", ["direct", "doubling"])
@pytest.mark.parametrize("name", ["long", "long_pattern", "graph_2048", "graph_32768", "grid"])
def test_shared_launches_give_the_bits_of_single_blocks(ctx, name, form):  # noqa: F811
    from paper_2103_10516_amd import mlct

    if name.startswith("graph"):
        g = wl.chung_lu(int(name.split("_")[1]), seed=5)
    else:
        g = wl.laplacian_2d(90) if name == "grid" else _matrix(name == "long_pattern")
    b = float(np.abs(g.to_scipy()).sum(axis=1).max()) + 1.0  # Gershgorin
    op = _op(ctx, g)
    mode = mlct.MLCT_DIRECT if form == "direct" else mlct.MLCT_DOUBLING
    for degrees, m, saves in LEVELS:
        args = (mlct.MLCT_CUBE, -b, b, degrees, m, 9, mlct.MLCT_FP32, mode)
        want, shared = _estimate(ctx, op, *args, alone=True)
        assert not shared
        got, shared = _estimate(ctx, op, *args)
        if form == "doubling":
            assert shared == saves, (degrees, m)
        _same(got, want)
        item = dict(op=op, kind=mlct.MLCT_CUBE, a=-b, b=b, degrees=degrees, m=m, seed=9)
        for launch in (mlct.MLCT_BATCH_LOCKSTEP, mlct.MLCT_BATCH_PERSISTENT):
            for r in mlct.mlct_estimate_batch(ctx, [item, item], mlct.MLCT_FP32, mode | launch):
                _same({**want, **r}, want)
    op.close()


def test_errors_are_those_of_single_blocks(ctx):  # noqa: F811
    from paper_2103_10516_amd import mlct

    op = _op(ctx, wl.laplacian_2d(20))
    for a, b, degrees, m in ((1.0, 2.0, [8, 20], [128, 64]), (1.0, 2.0, [20, 8], [128, 64]),
                             (1.0, 2.0, [8, 20], [128, 0]), (2.0, 1.0, [8, 20], [128, 64])):
        text = []
        for alone in (True, False):
            with pytest.raises(mlct.MlctError) as e:
                _estimate(ctx, op, mlct.MLCT_LOG, a, b, degrees, m, 3, mlct.MLCT_FP32,
                          mlct.MLCT_DOUBLING, alone=alone)
            text.append(str(e.value))
        assert text[0] == text[1]
    op.close()
