"""A pattern of INT32_MAX entries, the most an operator takes: its last rows, a
short one and a chunked one that ends at the last index, beside rows of 255
entries.  Every row's columns are one interval, so that the oracle's products
are differences of prefix sums."""
import numpy as np
import pytest

from oracle import lanczos, probes

pytestmark = pytest.mark.gpu

NNZ = 2**31 - 1
W = 255
LEAD = 8  # rows of one entry, which put the last rows into one wave's 16
MAIN = (NNZ - LEAD - 1 - 300) // W  # rows of W entries; then one of 1 and the rest
LAST = NNZ - LEAD - 1 - W * MAIN
D = LEAD + MAIN + 2


class Intervals:
    """A x from prefix sums."""

    def __init__(self, lo, n):
        self.lo, self.n = lo, n

    def __matmul__(self, x):
        # 80-bit sums: a float64 prefix sum of 8 M terms would lose 4 digits
        wide = np.int64 if x.dtype == np.int64 else np.longdouble
        p = np.concatenate([[wide(0)], np.cumsum(x, dtype=wide)])
        return (p[self.lo + self.n] - p[self.lo]).astype(x.dtype)


@pytest.fixture(scope="module")
def operator():
    import torch

    from paper_2103_10516_amd import mlct

    assert 300 <= LAST < 300 + W and D % 16 >= 4
    n = np.full(D, W, dtype=np.int64)
    n[:LEAD] = 1
    n[-2:] = [1, LAST]
    lo = np.clip(np.arange(D) - W // 2, 0, D - W)
    lo[-2:] = [5, D - LAST]
    rowptr = np.concatenate([[0], np.cumsum(n)])
    assert rowptr[-1] == NNZ
    col = torch.empty(NNZ, dtype=torch.int32, device="cuda")
    first = torch.from_numpy(lo.astype(np.int32)).cuda()
    step = torch.arange(W, dtype=torch.int32, device="cuda")
    col[:LEAD] = first[:LEAD]
    for a in range(LEAD, LEAD + MAIN, 1 << 20):
        b = min(a + (1 << 20), LEAD + MAIN)
        col[rowptr[a]:rowptr[b]] = (first[a:b, None] + step).reshape(-1)
    col[rowptr[D - 2]] = 5
    col[rowptr[D - 1]:] = torch.arange(D - LAST, D, dtype=torch.int32, device="cuda")
    ctx = mlct.mlct_create(0)
    op = mlct.mlct_op_csr(ctx, torch.from_numpy(rowptr.astype(np.int32)).cuda(), col)
    yield ctx, op, Intervals(lo, n)
    op.close()
    ctx.close()


def test_lanczos(operator):
    from paper_2103_10516_amd import mlct

    ctx, op, A = operator
    al, be, _ = mlct.mlct_lanczos(ctx, op, 4, 11, 0.01)
    oa, ob = lanczos.lanczos(A, D, 4, 11)
    # the tolerances of the other parity tests of the tridiagonal
    np.testing.assert_allclose(al, oa, rtol=1e-9, atol=1e-9 * np.max(np.abs(oa)))
    np.testing.assert_allclose(be, ob, rtol=1e-9, atol=1e-9 * np.max(np.abs(ob)))


def test_triangles(operator):
    from paper_2103_10516_amd import mlct

    ctx, op, A = operator
    _, w = mlct.mlct_triangles(ctx, op, 2, 7)
    for p, z in enumerate(probes.rademacher(D, np.arange(2), 7).astype(np.int64)):
        y = A @ z
        np.testing.assert_array_equal(w[p], [(z * y).sum(), (y * y).sum(), (y * (A @ y)).sum()])
