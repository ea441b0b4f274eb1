"""Rows past the straight-line capacity: the slots' chunk edges (4, 8, 16
entries), rows at the chunked sum's limit (256) and past it, several such
rows in one band, and one with more chunks than a workgroup has slots."""
import numpy as np
import pytest

from oracle import cheb, moments, probes
from paper_2103_10516_amd import workloads as wl
from tests.tolerances import U64, fp_moment_tol, kappa_csr, moment_tol, rho_rows

pytestmark = pytest.mark.gpu

LENGTHS = [0, 1, 3, 4, 5, 8, 9, 12, 15, 16, 17, 31, 32, 33, 48, 255, 256, 257, 300, 511, 512, 513]
D = 10007  # a last group of rows that is not full
BIG = 8449  # 34 chunks: past the 32 slots of a workgroup in FP32, its last chunk one entry


def _matrix(pattern: bool) -> wl.CSR:
    """Symmetric, rows of every length of LENGTHS and BIG: row i < len(want)
    has want[i] entries, all in the columns past the wanted rows."""
    rng = np.random.default_rng(3)
    want = [BIG] + LENGTHS * 3
    k = len(want)
    r, c = [], []
    for i, n in enumerate(want):
        r.append(np.full(n, i))
        c.append(k + rng.permutation(D - k)[:n])
    r, c = np.concatenate(r), np.concatenate(c)
    v = rng.uniform(-1.0, 1.0, size=r.size).astype(np.float32)
    R, C, Vv = np.concatenate([r, c]), np.concatenate([c, r]), np.concatenate([v, v])
    order = np.lexsort((C, R))
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(R, minlength=D))])
    g = wl.CSR(D, rowptr.astype(np.int32), C[order].astype(np.int32),
               None if pattern else Vv[order])
    assert set(want) <= set(np.diff(g.rowptr)[:k])
    return g


@pytest.fixture(scope="module")
def ctx():
    import torch

    from paper_2103_10516_amd import mlct

    assert torch.cuda.is_available()
    c = mlct.mlct_create(0)
    yield c
    c.close()


@pytest.mark.parametrize("pattern", [False, True])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_long_rows_match_oracle(ctx, pattern, prec):
    import torch

    from paper_2103_10516_amd import mlct

    g = _matrix(pattern)
    A = g.to_scipy()
    b = float(np.abs(A).sum(axis=1).max()) + 1.0  # Gershgorin
    n, m, seed, first = 24, 70, 5, 3
    op = mlct.mlct_op_csr(ctx, torch.from_numpy(g.rowptr).cuda(), torch.from_numpy(g.col).cuda(),
                          None if g.val is None else torch.from_numpy(g.val).cuda())
    P = mlct.MLCT_FP64 if prec == "fp64" else mlct.MLCT_FP32
    Z = probes.rademacher(g.d, np.arange(first, first + m), seed).T
    alpha, beta = cheb.affine_map(-b, b)
    want = moments.moments_direct(A, Z, alpha, beta, n)
    rn, kappa = int(np.max(np.diff(g.rowptr))), kappa_csr(g, alpha, beta)
    got = {}
    for mode in (mlct.MLCT_DIRECT, mlct.MLCT_DOUBLING):
        tol = (moment_tol(n, g.d, U64, rn, kappa) if prec == "fp64" else
               fp_moment_tol(n, g.d, "fp32", rn, rho_rows(A), kappa, alpha, beta,
                             mode == mlct.MLCT_DOUBLING))
        got[mode] = mlct.mlct_moments(ctx, op, -b, b, n, mlct.rademacher_probes(seed, m, first),
                                      P, mode)
        assert np.max(np.abs(got[mode] - want) / tol[None, :]) <= 1.0
    # explicit probes with the same signs give the same bits
    ex = mlct.explicit_probes(torch.from_numpy(Z.astype(np.int8)).cuda())
    assert np.array_equal(mlct.mlct_moments(ctx, op, -b, b, n, ex, P, mlct.MLCT_DIRECT),
                          got[mlct.MLCT_DIRECT])
    if prec == "fp32":  # the batched launches give the single call's bits
        item = dict(op=op, kind=mlct.MLCT_CUBE, a=-b, b=b, degrees=[6, 24], m=[70, 20], seed=9)
        one = mlct.mlct_estimate(ctx, op, mlct.MLCT_CUBE, -b, b, [6, 24], [70, 20], 9,
                                 mlct.MLCT_FP32, mlct.MLCT_DIRECT)
        for form in (mlct.MLCT_BATCH_LOCKSTEP, mlct.MLCT_BATCH_PERSISTENT):
            r = mlct.mlct_estimate_batch(ctx, [item, dict(item, seed=10)], mlct.MLCT_FP32,
                                         mlct.MLCT_DIRECT | form)[0]
            assert r["value"] == one["value"]
            assert np.array_equal(r["level_var"], one["level_var"])
    op.close()
