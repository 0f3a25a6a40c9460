"""GPU: the coarsest level's dense inverse at the edges of its panels (16
columns, 8 from 1,537 rows on), of the rows a thread holds (512 each) and of
its tiles (64 x 128), with row interchanges in every column, and on an
ill-conditioned diffusion matrix.

A single field of at most coarse_max rows is solved by that inverse alone:
apply(r) = A^-1 r.  Bound: an explicit inverse computed with partial pivoting
is accurate to a modest multiple of n u kappa(A); 8 n u kappa is allowed.
"""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu


def _interchanges(n):
    """P (3 I + R) + 1e-3 I: small diagonal entries, well conditioned."""
    rng = np.random.default_rng(n)
    P = sp.csr_matrix((np.ones(n), (np.arange(n), rng.permutation(n))), shape=(n, n))
    R = sp.random(n, n, density=min(1.0, 6.0 / n), random_state=rng, format="csr")
    return (P @ (3.0 * sp.eye(n) + R) + 1e-3 * sp.eye(n)).toarray()


def _diffusion(m):
    """m x m cells, permeabilities over four decades, held at one corner."""
    k = 1e4 ** np.random.default_rng(m).random((m, m))
    A = np.zeros((m * m, m * m))
    for i in range(m):
        for j in range(m):
            for a, b in ((i, j + 1), (i + 1, j)):
                if a < m and b < m:
                    t = 2 * k[i, j] * k[a, b] / (k[i, j] + k[a, b])
                    p, q = i * m + j, a * m + b
                    A[p, p] += t
                    A[q, q] += t
                    A[p, q] -= t
                    A[q, p] -= t
    A[0, 0] += 1.0
    return A


@pytest.mark.parametrize("make,n", [(_interchanges, n) for n in (
    2, 15, 16, 18, 31, 33, 63, 64, 65, 127, 129, 511, 512, 513, 1024, 1025, 1536, 1537, 1544, 2047)] +
    [(_diffusion, 9), (_diffusion, 30)])
def test_dense_inverse(make, n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_13079_amd as H
    A = make(n)
    n = A.shape[0]
    pat = sp.csr_matrix(((A != 0) | (A.T != 0)).astype(float))
    pat.sort_indices()
    rows = np.repeat(np.arange(n), np.diff(pat.indptr))
    dev = torch.device("cuda:0")
    rp, ci, v, fl = (torch.from_numpy(a).to(dev) for a in (
        pat.indptr.astype(np.int32), pat.indices.astype(np.int32), A[rows, pat.indices], np.zeros(n, np.int32)))
    g = H.Solver(rp, ci, v, fl, 1, [-1, 0, -2], coarse_max=max(n, 16), precision=0)
    x = np.random.default_rng(7).standard_normal(n)
    kappa = np.linalg.norm(A, 1) * np.linalg.norm(np.linalg.inv(A), 1)
    for M, tr in ((A, False), (A.T, True)):
        b = (M.astype(np.longdouble) @ x).astype(np.float64)
        z = g.apply(torch.from_numpy(b).to(dev), transpose=tr).cpu().numpy()
        err = np.abs(z - x).max() / np.abs(x).max()
        assert err <= 8 * n * 2.0 ** -53 * kappa, (n, tr, err, kappa)
