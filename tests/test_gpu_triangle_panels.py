"""Triangle moments over every number of 64-probe panels in a group, on
patterns with rows at the chunk edges, diagonal and repeated entries, sorted
or not, symmetric or not: exact integers, compared with int64 sums."""
import numpy as np
import pytest
import scipy.sparse as sp

from oracle import probes
from paper_2103_10516_amd import workloads as wl

pytestmark = pytest.mark.gpu

D = 3001


@pytest.fixture(scope="module")
def ctx():
    import torch

    from paper_2103_10516_amd import mlct

    assert torch.cuda.is_available()
    c = mlct.mlct_create(0)
    yield c
    c.close()


def _pattern(symmetric: bool, ordered: bool) -> wl.CSR:
    rng = np.random.default_rng(17)
    want = [0, 1, 4, 5, 8, 9, 15, 16, 17, 32, 33, 255, 256, 257, 512, 513, 2900]
    k = len(want)
    r = np.concatenate([np.full(n, i) for i, n in enumerate(want)]).astype(np.int64)
    c = np.concatenate([k + rng.permutation(D - k)[:n] for n in want]).astype(np.int64)
    # a random part with repeated entries, and diagonal entries (some twice)
    er, ec = rng.integers(k, D, size=(2, 9000))
    r, c = np.concatenate([r, er]), np.concatenate([c, ec])
    if symmetric:
        r, c = np.concatenate([r, c]), np.concatenate([c, r])
    dg = np.concatenate([rng.integers(0, D, size=50), [12, 12, 16, 16, 16]])
    r, c = np.concatenate([r, dg]), np.concatenate([c, dg])
    order = np.lexsort((c if ordered else rng.permutation(c.size), r))
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(r, minlength=D))])
    return wl.CSR(D, rowptr.astype(np.int32), c[order].astype(np.int32), None)


def _want(g, Z):
    A = sp.csr_matrix((np.ones(g.nnz, dtype=np.int64), g.col, g.rowptr), shape=(g.d, g.d))
    y = A @ Z
    return np.stack([(Z * y).sum(0), (y * y).sum(0), (y * (A @ y)).sum(0)], axis=1)


@pytest.mark.parametrize("symmetric,ordered", [(True, True), (True, False), (False, True)])
def test_every_panel_count(ctx, symmetric, ordered):
    import torch

    from paper_2103_10516_amd import mlct

    g = _pattern(symmetric, ordered)
    op = mlct.mlct_op_csr(ctx, torch.from_numpy(g.rowptr).cuda(), torch.from_numpy(g.col).cuda())
    for m in (1, 63, 64, 65, 128, 150, 256, 300, 512, 513, 700):
        res, w = mlct.mlct_triangles(ctx, op, m, 40 + m)
        Z = probes.rademacher(g.d, np.arange(m), 40 + m).T.astype(np.int64)
        want = _want(g, Z)
        np.testing.assert_array_equal(w, want, err_msg=f"m = {m}")
        assert res["sum_w3"] == want[:, 2].sum()
    op.close()


def test_one_panel_under_a_workspace_limit():
    """A limit that holds one panel and no more: the same results."""
    import torch

    from paper_2103_10516_amd import mlct

    g = _pattern(True, True)
    out = []
    for limited in (False, True):
        c = mlct.mlct_create(0)
        op = mlct.mlct_op_csr(c, torch.from_numpy(g.rowptr).cuda(), torch.from_numpy(g.col).cuda())
        if limited:
            mlct.mlct_set_workspace_limit(c, D * 8 + 2 * D * 128)
        out.append(mlct.mlct_triangles(c, op, 300, 5))
        c.close()
    np.testing.assert_array_equal(out[0][1], out[1][1])
    assert out[0][0] == out[1][0]
