"""Memory that only makes a call faster (packed dense operands, triangle panels
past the first, shared launches of small estimates) does not stand in the way of
a later call under a workspace limit, and goes back when one is set."""
import numpy as np
import pytest

from paper_2103_10516_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _op(ctx, g):
    import torch

    from paper_2103_10516_amd import mlct

    return mlct.mlct_op_csr(ctx, *(None if x is None else torch.from_numpy(x).cuda()
                                   for x in (g.rowptr, g.col, g.val)))


def _triangles(ctx, keep):
    from paper_2103_10516_amd import mlct

    keep.append(_op(ctx, wl.chung_lu(8000, seed=3)))
    mlct.mlct_triangles(ctx, keep[-1], 512, 5)


def _small_estimate(ctx, keep):
    from paper_2103_10516_amd import mlct

    keep.append(_op(ctx, wl.laplacian_2d(45)))
    mlct.mlct_timing(ctx, True)
    mlct.mlct_estimate(ctx, keep[-1], mlct.MLCT_LOG, 0.01, 8.01, [8, 20], [128, 64], 3,
                       mlct.MLCT_FP32, mlct.MLCT_DOUBLING)
    mlct.mlct_timing(ctx, False)
    assert mlct.mlct_timing_read(ctx, mlct.MLCT_KERNEL_BATCH_STEP)[0] > 0


G = wl.laplacian_2d(100)


def _later(limit, first=None):
    """FP64 moments of 10,000 rows under the limit, after another call or alone."""
    from paper_2103_10516_amd import mlct

    ctx, keep = mlct.mlct_create(0), []
    op = _op(ctx, G)
    mlct.mlct_set_workspace_limit(ctx, limit)
    try:
        if first:
            first(ctx, keep)
        return mlct.mlct_moments(ctx, op, 0.01, 8.01, 8, mlct.rademacher_probes(5, 64),
                                 mlct.MLCT_FP64, mlct.MLCT_DOUBLING)
    finally:
        for o in keep + [op]:
            o.close()
        ctx.close()


@pytest.mark.parametrize("first", [_triangles, _small_estimate])
def test_later_call_under_a_limit(first):
    from paper_2103_10516_amd import mlct

    lo, hi = 0, 1 << 26  # the least limit under which the later call runs alone
    while hi - lo > 4096:
        mid = (lo + hi) // 2
        try:
            want = _later(mid)
            hi = mid
        except mlct.MlctError as e:
            assert e.status == mlct.MLCT_ENOMEM
            lo = mid
    # slots that the first call alone uses: results, indices, small tables
    np.testing.assert_array_equal(_later(hi + (600 << 10), first), want)


def test_packed_operands_go_back_under_a_smaller_limit():
    import torch

    from paper_2103_10516_amd import mlct

    d = 8000  # 256 MB of packed FP32
    A = torch.full((d, d), 1.0 / d, device="cuda")
    ctx = mlct.mlct_create(0)
    op = mlct.mlct_op_dense(ctx, A)
    pr = mlct.rademacher_probes(5, 32)
    run = lambda: mlct.mlct_moments(ctx, op, -1.5, 1.5, 20, pr, mlct.MLCT_FP32,  # noqa: E731
                                    mlct.MLCT_DOUBLING)
    first = run()
    held = torch.cuda.mem_get_info()[0]
    mlct.mlct_set_workspace_limit(ctx, 1 << 28)
    assert torch.cuda.mem_get_info()[0] - held >= 4 * d * d
    mlct.mlct_set_workspace_limit(ctx, 0)
    np.testing.assert_array_equal(run(), first)
    op.close()
    ctx.close()
