"""GPU: the rows of a transposed matrix are in column order, entry by entry.

R = P^T of a two-level hierarchy, whose row for a hub's aggregate has as many
entries as the hub has neighbours: on both sides of the edges of the sort (64
entries per pass of a wavefront, 256 for the wavefront, 2,048 for a block).
R's pattern and values are compared bitwise with P^T, sorted on the host.
"""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("length", [2, 5, 63, 64, 65, 127, 128, 129, 255, 256, 257, 600, 2047, 2048, 2049, 2600])
def test_restriction_is_the_sorted_transpose(length):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_13079_amd as H
    # stars of `length` rows, the hubs spread over the numbering; each hub's star is one aggregate, and a star's rows
    # only meet each other, so P's column of an aggregate has the star's rows
    stars = max(2, 3000 // length)
    n = stars * length
    rng = np.random.default_rng(length)
    rows = rng.permutation(n).reshape(stars, length)
    hub, leaf = np.repeat(rows[:, 0], length - 1), rows[:, 1:].ravel()
    w = -1.0 - rng.random(hub.size)
    A = sp.coo_matrix((np.concatenate([w, w]), (np.concatenate([hub, leaf]), np.concatenate([leaf, hub]))), shape=(n, n))
    A = (A + sp.diags(1.0 - np.asarray(A.sum(axis=1)).ravel())).tocsr()
    A.sort_indices()
    dev = torch.device("cuda:0")
    rp, ci, v, fl = (torch.from_numpy(a).to(dev) for a in (
        A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data, np.zeros(n, np.int32)))
    g = H.Solver(rp, ci, v, fl, 1, [-1, 0, -2], coarse_max=stars, precision=0, theta=[0.0])
    p = g.get_level(0, 0, "P")
    P = sp.csr_matrix((p[2], p[1], p[0]), shape=(n, p[3]))
    T = P.T.tocsr()
    T.sort_indices()
    r = g.get_level(0, 0, "R")
    assert T.shape == (stars, n) and np.diff(T.indptr).max() == length
    assert np.array_equal(r[0], T.indptr) and np.array_equal(r[1], T.indices)
    assert np.array_equal(r[2].view(np.int64), T.data.view(np.int64))
