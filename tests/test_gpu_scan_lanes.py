"""GPU: setup passes that take one thread per row where rows are short, and
groups of lanes where the longest exceeds 24 entries: hierarchies bitwise the
oracle's on both sides of that, on grids with one long row and on stars whose
coarse levels have long rows too."""
import numpy as np
import pytest
import scipy.sparse as sp

import oracle

pytestmark = pytest.mark.gpu


def _grid_with_hub(longest, m=36):
    """m x m five-point grid; one row gets neighbours until it has `longest` entries."""
    n = m * m
    rng = np.random.default_rng(longest)
    i = np.arange(n).reshape(m, m)
    e = [np.stack([i[:, :-1].ravel(), i[:, 1:].ravel()]), np.stack([i[:-1].ravel(), i[1:].ravel()])]
    hub = n // 2 + m // 2
    others = np.setdiff1d(np.arange(n), [hub, hub - 1, hub + 1, hub - m, hub + m])
    far = rng.choice(others, longest - 5, replace=False)
    e.append(np.stack([np.full(far.size, hub), far]))
    p, q = np.concatenate(e, axis=1)
    w = -0.5 - rng.random(p.size)
    A = sp.coo_matrix((np.concatenate([w, w]), (np.concatenate([p, q]), np.concatenate([q, p]))), shape=(n, n))
    A = (A + sp.diags(0.05 - 1.1 * np.asarray(A.sum(axis=1)).ravel())).tocsr()
    A.sort_indices()
    assert np.diff(A.indptr).max() == longest and A.nnz / n <= 7.5
    return A


@pytest.mark.parametrize("theta", [0.0, 0.25])
@pytest.mark.parametrize("longest", [5, 8, 9, 23, 24, 25, 32, 33, 90])
def test_hierarchy_bit_exact(longest, theta):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_13079_amd as H
    A = _grid_with_hub(longest)
    n = A.shape[0]
    arrays = A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data, np.zeros(n, np.int32)
    opt = dict(coarse_max=16, theta=[theta], precision=0)
    rp, ci, v, fl = (torch.from_numpy(a).to("cuda:0") for a in arrays)
    g = H.Solver(rp, ci, v, fl, 1, [-1, 0, -2], **opt)
    o = oracle.Oracle(arrays[0], arrays[1], arrays[2], 1, arrays[3], [-1, 0, -2], **opt).amg(0)
    levels = g.stats()["levels"][0]
    assert levels == o.levels and levels > 2
    for l in range(levels):
        coarsest = l + 1 == levels
        for w in ("A", "AT") if coarsest else ("A", "P", "R", "AT"):
            got, want = g.get_level(0, l, w), o.get(l, w)
            assert got[3] == want[3] and np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1]), (l, w)
            assert np.array_equal(got[2].view(np.int64), want[2].view(np.int64)), (l, w)
        if not coarsest:
            agg, scalars = g.aggregates(0, l)
            assert np.array_equal(agg, o.agg(l)) and scalars == o.scalars(l), l
