"""The passes over the Lanczos basis at the edges of their column pieces (16,
32, 64 columns in registers, more in two pieces) and of their row tiles, on
rows of every length class of the product, against the FP64 oracle."""
import numpy as np
import pytest

from oracle import lanczos
from paper_2103_10516_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _matrix(d: int) -> wl.CSR:
    """Random symmetric rows plus one of 300 entries (chunked) and empty ones;
    a spread diagonal keeps 128 steps from converging."""
    import scipy.sparse as sp

    rng = np.random.default_rng(d)
    A = sp.random(d, d, density=min(0.5, 9.0 / d), random_state=rng, dtype=np.float64)
    hub = sp.coo_matrix((rng.uniform(-1, 1, 300), (np.full(300, 7), rng.permutation(d)[:300])),
                        shape=(d, d)) if d > 400 else sp.coo_matrix((d, d))
    A = A + hub
    A = (A + A.T + sp.diags(np.where(np.arange(d) % 50 == 3, 0.0, rng.uniform(-40, 40, d)))).tocsr()
    A.eliminate_zeros()
    A.sort_indices()
    return wl.CSR(d, A.indptr.astype(np.int32), A.indices.astype(np.int32),
                  A.data.astype(np.float32))


@pytest.mark.parametrize("d", [130, 4097, 70001])
def test_basis_passes_match_oracle(d):
    import torch

    from paper_2103_10516_amd import mlct

    g = _matrix(d)
    ctx = mlct.mlct_create(0)
    op = mlct.mlct_op_csr(ctx, *(torch.from_numpy(x).cuda() for x in (g.rowptr, g.col, g.val)))
    A = g.to_scipy()
    for steps in (1, 15, 16, 17, 32, 33, 64, 65, 128):
        al, be, info = mlct.mlct_lanczos(ctx, op, steps, 11, 0.01)
        oa, ob = lanczos.lanczos(A, d, steps, 11)
        assert len(al) == len(oa) == steps
        # the tolerances of the other parity tests of the tridiagonal
        np.testing.assert_allclose(al, oa, rtol=1e-9, atol=1e-9 * np.max(np.abs(oa)))
        np.testing.assert_allclose(be, ob, rtol=1e-9, atol=1e-9 * np.max(np.abs(ob)))
        if steps > 1:
            T = np.diag(oa) + np.diag(ob[:-1], 1) + np.diag(ob[:-1], -1)
            th = np.linalg.eigvalsh(T)
            assert info["theta_min"] == pytest.approx(th[0], rel=1e-9)
            assert info["theta_max"] == pytest.approx(th[-1], rel=1e-9)
    ctx.close()
