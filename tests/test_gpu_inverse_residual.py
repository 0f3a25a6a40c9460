"""GPU: the coarsest level's dense inverse X leaves residuals ||b - A X b|| as
small as LU with substitution, also where the rows of A differ in scale, in
both directions, for panels of 16 columns and (from 1,537 rows on) of 8.

Each column of X is one forward and one backward substitution with the factors
of a partially pivoted LU, so |b - A X b| <= c n u |L| |U| |X| |b| row by row,
with the same c as for scipy's.  The two differ in the order of their sums
only: a factor of 10 between the two residuals is allowed.
"""
import numpy as np
import pytest
import scipy.linalg as sl
import scipy.sparse as sp

pytestmark = pytest.mark.gpu


def _diffusion(m, seed):
    """m x m cells, permeabilities over four decades, held at one corner."""
    k = 1e4 ** np.random.default_rng(seed).random((m, m))
    i = np.arange(m * m).reshape(m, m)
    rows, cols, vals = [], [], []
    for p, q, a, b in ((i[:, :-1], i[:, 1:], k[:, :-1], k[:, 1:]), (i[:-1], i[1:], k[:-1], k[1:])):
        t, p, q = (2 * a * b / (a + b)).ravel(), p.ravel(), q.ravel()
        rows += [p, q, p, q]
        cols += [p, q, q, p]
        vals += [t, t, -t, -t]
    A = sp.coo_matrix((np.concatenate(vals), (np.concatenate(rows), np.concatenate(cols)))).tocsr()
    A[0, 0] += 1.0
    return A


def _solver(A, **opt):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_13079_amd as H
    A = A.tocsr()
    A.sort_indices()
    dev = torch.device("cuda:0")
    rp, ci, v, fl = (torch.from_numpy(a).to(dev) for a in (
        A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data, np.zeros(A.shape[0], np.int32)))
    return H.Solver(rp, ci, v, fl, 1, [-1, 0, -2], coarse_max=max(A.shape[0], 16), precision=0, **opt)


@pytest.mark.parametrize("m", [7, 20, 40])
@pytest.mark.parametrize("span", [0, 4, 8])
def test_residual_at_the_level_of_lu(m, span):
    import torch
    rng = np.random.default_rng(100 * m + span)
    A = sp.diags(10.0 ** (span * rng.random(m * m))) @ _diffusion(m, m)
    D = A.toarray()
    X = sl.lu_solve(sl.lu_factor(D), np.eye(m * m))
    g = _solver(A)
    b = rng.standard_normal(m * m)
    for M, Xl, tr in ((D, X, False), (D.T, X.T, True)):
        Ml = M.astype(np.longdouble)
        got, ref = (np.linalg.norm((b - Ml @ z.astype(np.longdouble)).astype(np.float64)) for z in (
            g.apply(torch.from_numpy(b).cuda(), transpose=tr).cpu().numpy(), Xl @ b))
        assert got <= 10 * ref, (m, span, tr, got, ref)


@pytest.mark.parametrize("value", [2.0 ** -1050, float("inf")])
def test_extreme_pivots_are_factored(value):
    """Only a column of zeros makes the matrix singular: pivots whose high word
    is zero and infinite ones are taken (new values are not checked)."""
    import torch
    n = 33
    A = sp.diags([np.full(n - 1, -1.0), np.full(n, 4.0), np.full(n - 1, -1.0)], [-1, 0, 1]).tocsr()
    A.sort_indices()
    g = _solver(A)
    v = A.copy()
    for j in (n - 2, n - 1):  # the last row's off-diagonal entries go, its diagonal is the last pivot
        v[n - 1, j] = 0.0 if j < n - 1 else value
        v[j, n - 1] = 0.0 if j < n - 1 else value
    assert v.nnz == A.nnz
    g.set_values(torch.from_numpy(v.data).cuda())
    z = g.apply(torch.zeros(n, dtype=torch.float64, device="cuda"))
    assert z.shape == (n,)
