"""Triangle moments whose first product leaves 16 bits in some panels of a group
and not in others: exact integers for every number of panels."""
import numpy as np
import pytest
import scipy.sparse as sp

from oracle import probes
from paper_2103_10516_amd import workloads as wl
from tests.test_gpu_triangle_panels import _want, ctx  # noqa: F401

pytestmark = pytest.mark.gpu

D = 700
ROWS = [(3, np.arange(40, 48)), (350, np.arange(100, 108)), (699, np.arange(200, 209))]
TIMES = 4100  # entries per column: 8 equal signs make 32,800


def _pattern(symmetric: bool) -> wl.CSR:
    rng = np.random.default_rng(5)
    r = [np.full(len(c) * TIMES, i) for i, c in ROWS]
    c = [np.repeat(c, TIMES) for _, c in ROWS]
    er, ec = rng.integers(0, D, size=(2, 3000))
    r, c = np.concatenate(r + [er]), np.concatenate(c + [ec])
    if symmetric:
        r, c = np.concatenate([r, c]), np.concatenate([c, r])
    order = np.lexsort((c, r))
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(r, minlength=D))])
    return wl.CSR(D, rowptr.astype(np.int32), c[order].astype(np.int32), None)


@pytest.mark.parametrize("symmetric", [True, False])
def test_escapes_in_some_panels(ctx, symmetric):  # noqa: F811
    import torch

    from paper_2103_10516_amd import mlct

    g = _pattern(symmetric)
    op = mlct.mlct_op_csr(ctx, torch.from_numpy(g.rowptr).cuda(), torch.from_numpy(g.col).cuda())
    A = sp.csr_matrix((np.ones(g.nnz, dtype=np.int64), g.col, g.rowptr), shape=(D, D))
    seen = set()
    for m, seed in ((64, 1), (100, 2), (192, 3), (300, 4), (320, 5), (448, 6), (512, 7), (700, 8),
                    (512, 9), (512, 10)):
        _, w = mlct.mlct_triangles(ctx, op, m, seed)
        Z = probes.rademacher(D, np.arange(m), seed).T.astype(np.int64)
        np.testing.assert_array_equal(w, _want(g, Z), err_msg=f"m = {m}")
        past = (np.abs(A @ Z) > 32767).any(axis=0)
        seen |= {(p % 8, bool(past[64 * p:64 * p + 64].any())) for p in range((m + 63) // 64)}
    # every panel of a group with and without values past 16 bits
    assert seen == {(p, e) for p in range(8) for e in (False, True)}
    op.close()
