"""Dense matrices on both sides of the steps from which a block is packed:
by rows (96, 128, 160), probes (32, 64, 128 of the padded block) and steps."""
import numpy as np
import pytest

from oracle import cheb, moments, probes
from tests.test_gpu_dense import _prec, _tol, ctx  # noqa: F401
from tests.test_gpu_dense_packed import A0, B0, _device, _matrix

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("d", [95, 96, 127, 128, 159, 160])
def test_moments_on_both_sides(ctx, prec, d):  # noqa: F811
    from paper_2103_10516_amd import mlct

    A = _matrix(d)
    op = mlct.mlct_op_dense(ctx, _device(A, prec))
    alpha, beta = cheb.affine_map(A0, B0)
    Aop = A if prec == "fp64" else A.astype(np.float32).astype(np.float64)
    for m in (32, 33, 97):
        Z = probes.rademacher(d, np.arange(m), 9).T
        for n in (3, 4, 5, 6, 7, 9, 10):
            got = mlct.mlct_moments(ctx, op, A0, B0, n, mlct.rademacher_probes(9, m), _prec(prec),
                                    mlct.MLCT_DIRECT)
            want = moments.moments_direct(Aop, Z, alpha, beta, n)
            tol = _tol(prec, n, d, Aop, alpha, beta, False)
            assert np.all(np.abs(got - want) <= tol[None, :]), (m, n)
    op.close()


def test_few_probes_of_a_large_matrix(ctx):  # noqa: F811
    """FP32, up to 32 probes from 8,192 rows on: by rows at four steps, packed at
    five."""
    from paper_2103_10516_amd import mlct

    d, m = 8192, 20
    A = np.random.default_rng(5).standard_normal((d, d), dtype=np.float32)
    A = (A + A.T) / np.float32(np.sqrt(2.0 * d))  # spectrum near [-2, 2]
    op = mlct.mlct_op_dense(ctx, _device(A, "fp32"))
    alpha, beta = cheb.affine_map(-2.5, 2.5)
    Aop = A.astype(np.float64)
    want = moments.moments_direct(Aop, probes.rademacher(d, np.arange(m), 9).T, alpha, beta, 5)
    tol = _tol("fp32", 5, d, Aop, alpha, beta, False)
    for n in (4, 5):
        got = mlct.mlct_moments(ctx, op, -2.5, 2.5, n, mlct.rademacher_probes(9, m), _prec("fp32"),
                                mlct.MLCT_DIRECT)
        assert np.all(np.abs(got - want[:, :n + 1]) <= tol[None, :n + 1]), n
    op.close()
