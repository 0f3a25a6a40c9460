"""GPU: rows of a transposed matrix are put in column order by one wavefront
up to 256 entries (64 per pass) and by a block beyond: lengths on both sides
of those edges, through the adjoint solve, which reads A^T.

Each matrix has a column of the given length among short ones.  The bound is
the solver's own: a true relative residual of 1e-8 (plus the rounding of
forming it here, below 1e-12); a lost, doubled or misplaced entry of the long
column is of the order of 1e-2.
"""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("length", [1, 2, 4, 5, 63, 64, 65, 127, 128, 129, 255, 256, 257, 600])
def test_transposed_rows(length):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_13079_amd as H
    n = 640
    rng = np.random.default_rng(length)
    others = 1 + rng.permutation(n - 1)[:length - 1]
    A = sp.lil_matrix((n, n))
    A.setdiag(4.0)
    for i in others:
        A[i, 0] = 0.1 * (1 + rng.random())
        A[0, i] = 1e-3 * rng.random() + 1e-4
    A = sp.csr_matrix(A)
    A.sort_indices()
    dev = torch.device("cuda:0")
    rp, ci, v, fl = (torch.from_numpy(a).to(dev) for a in (
        A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data, np.zeros(n, np.int32)))
    g = H.Solver(rp, ci, v, fl, 1, [-1, 0, -2], coarse_max=n, precision=0)
    b = rng.standard_normal(n)
    x, status, _, _ = g.solve(torch.from_numpy(b).to(dev), transpose=True)
    res = np.linalg.norm(b - A.T @ x.cpu().numpy()) / np.linalg.norm(b)
    assert status == 0 and res <= 1e-8 + 1e-12, (length, status, res)
