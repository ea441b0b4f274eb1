"""Operators whose blocks exceed 4 GiB, where gathers take 64-bit addresses: rows
of every length class at both ends and past the 4 GiB line, on a chain of as many
rows as that takes.  The recurrence is checked with explicit probes that live on
those rows, so that the tolerance is that of a small operator."""
import numpy as np
import pytest

from oracle import cheb, moments, probes
from tests.tolerances import U64, fp_moment_tol, moment_tol

pytestmark = pytest.mark.gpu

LENGTHS = [9, 16, 17, 33, 255, 257, 600]
NORM = 2.0 + np.sqrt(600.0) + 2.0  # chain, largest star, the stars' few shared vertices


class Chain:
    """0/1 pattern of a path of d vertices with a star of each length of LENGTHS
    around vertices at the start, the middle and the end."""

    def __init__(self, d):
        rng = np.random.default_rng(d)
        self.d = d
        at = np.concatenate([3 + np.arange(7), d // 2 + np.arange(7), d - 8 + np.arange(7)])
        u = np.concatenate([np.full(n, i) for i, n in zip(at, LENGTHS * 3)])
        v = rng.integers(20, d - 20, u.size)
        self.u, self.v = np.concatenate([u, v]), np.concatenate([v, u])
        self.at = at

    def __matmul__(self, x):
        y = np.zeros_like(x)
        y[1:] += x[:-1]
        y[:-1] += x[1:]
        np.add.at(y, self.u, x[self.v])
        return y

    def csr(self):
        """rowptr, col on the device."""
        import torch

        i = torch.arange(self.d - 1, device="cuda")
        r = torch.cat([i, i + 1, torch.from_numpy(self.u).cuda()])
        c = torch.cat([i + 1, i, torch.from_numpy(self.v).cuda()])
        key = torch.sort(r * self.d + c)[0]
        n = torch.bincount(key // self.d, minlength=self.d)
        rowptr = torch.zeros(self.d + 1, dtype=torch.int64, device="cuda")
        rowptr[1:] = torch.cumsum(n, 0)
        return rowptr.int(), (key % self.d).int()

    def signs(self):
        """Three explicit probes on the stars' centres, their leaves and the ends."""
        rng = np.random.default_rng(1)
        Z = np.zeros((self.d, 3), dtype=np.int8)
        rows = np.unique(np.concatenate([self.u, np.arange(40), np.arange(self.d - 40, self.d)]))
        Z[rows] = rng.choice([-1, 1], (rows.size, 3))
        return Z


@pytest.fixture
def ctx():
    import torch

    from paper_2103_10516_amd import mlct

    assert torch.cuda.is_available()
    torch.cuda.empty_cache()
    c = mlct.mlct_create(0)
    yield c
    c.close()
    torch.cuda.empty_cache()


def _check(got, A, Z, a, b, n, prec, norm2, doubling):
    alpha, beta = cheb.affine_map(a, b)
    Z = Z.astype(np.float64)
    want = moments.moments_direct(A, Z, alpha, beta, n)
    for p in range(Z.shape[1]):
        z2 = float(Z[:, p] @ Z[:, p])
        # rows of up to 602 entries; |A_hat| at most 1 in the two-norm
        kappa = alpha * norm2 + abs(beta)
        tol = (moment_tol(n, z2, U64, 602, kappa) if prec == "fp64" else
               fp_moment_tol(n, z2, "fp32", 602, np.sqrt(602.0) * norm2, kappa, alpha, beta,
                             doubling))
        assert np.all(np.abs(got[p] - want[p]) <= tol), p


@pytest.mark.parametrize("valued", [False, True])
@pytest.mark.parametrize("prec,d", [("fp32", 2**24 + 5), ("fp64", 2**23 + 5)])
def test_moments(ctx, prec, d, valued):
    import torch

    from paper_2103_10516_amd import mlct

    A = Chain(d)
    rowptr, col = A.csr()
    val = torch.ones(col.numel(), device="cuda") if valued else None
    op = mlct.mlct_op_csr(ctx, rowptr, col, val)
    Z = A.signs()
    pr = mlct.explicit_probes(torch.from_numpy(Z).cuda())
    P = mlct.MLCT_FP64 if prec == "fp64" else mlct.MLCT_FP32
    for mode in (mlct.MLCT_DIRECT, mlct.MLCT_DOUBLING):
        got = mlct.mlct_moments(ctx, op, -NORM, NORM, 4, pr, P, mode)
        _check(got, A, Z, -NORM, NORM, 4, prec, NORM, mode == mlct.MLCT_DOUBLING)
    if prec == "fp64":  # two Lanczos steps integrate x^3 exactly
        got = mlct.mlct_slq_quadforms(ctx, op, mlct.MLCT_CUBE, 2, pr)
        X = Z.astype(np.float64)
        Y = A @ X
        np.testing.assert_allclose(got, np.einsum("ip,ip->p", Y, A @ Y), rtol=1e-9,
                                   atol=1e-9 * np.einsum("ip,ip->p", Y, Y).max())
    op.close()


class Gram:
    def __init__(self, X):
        self.X = X

    def __matmul__(self, x):
        return self.X @ (self.X @ x) + 0.5 * x  # X is symmetric


@pytest.mark.parametrize("prec,d", [("fp32", 2**24 + 5), ("fp64", 2**23 + 5)])
def test_gram_moments(ctx, prec, d):
    import torch

    from paper_2103_10516_amd import mlct

    X = Chain(d)
    rowptr, col = X.csr()
    op = mlct.mlct_op_gram_csr(ctx, rowptr, col, None, d, 0.5)
    Z = X.signs()
    pr = mlct.explicit_probes(torch.from_numpy(Z).cuda())
    P = mlct.MLCT_FP64 if prec == "fp64" else mlct.MLCT_FP32
    b = NORM**2 + 0.5
    got = mlct.mlct_moments(ctx, op, 0.0, b, 3, pr, P, mlct.MLCT_DOUBLING)
    _check(got, Gram(X), Z, 0.0, b, 3, prec, b, True)
    op.close()


def test_triangles(ctx):
    """Panels of 64 probes past 4 GiB: from 2^25 rows on."""
    from paper_2103_10516_amd import mlct

    d = 2**25 + 5
    A = Chain(d)
    op = mlct.mlct_op_csr(ctx, *A.csr())
    _, w = mlct.mlct_triangles(ctx, op, 2, 7)
    for p, z in enumerate(probes.rademacher(d, np.arange(2), 7).astype(np.int64)):
        y = A @ z
        np.testing.assert_array_equal(w[p], [(z * y).sum(), (y * y).sum(), (y * (A @ y)).sum()])
    op.close()
