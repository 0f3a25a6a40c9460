"""GPU: a value update whose rebuild fails leaves a context without a
preconditioner.  Every call that would read it returns an error (no launch),
and an update with valid values makes the context whole again."""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fields", [1, 3])
def test_failed_update(fields):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_13079_amd as H
    n = 40
    good = sp.block_diag([sp.diags([-1.0, 2.5, -1.0], [-1, 0, 1], shape=(n, n))] * fields).tocsr()
    good.sort_indices()
    bad = good.copy()
    r = n * (fields - 1)  # the last field: rows 0 and 1 become equal, its coarsest matrix singular
    for i, j in ((r, r), (r, r + 1), (r + 1, r), (r + 1, r + 1), (r + 1, r + 2), (r + 2, r + 1)):
        bad[i, j] = 1.0 if max(i, j) < r + 2 else 0.0
    assert bad.nnz == good.nnz
    dev = torch.device("cuda:0")

    def to(a):
        return torch.from_numpy(a).to(dev)
    g = H.Solver(to(good.indptr.astype(np.int32)), to(good.indices.astype(np.int32)), to(good.data),
                 to(np.repeat(np.arange(fields, dtype=np.int32), n)), fields, [-1, *range(fields), -2], coarse_max=64)
    b = to(good @ np.linspace(1.0, 2.0, n * fields))
    z, out = g.apply(b), torch.empty_like(b)
    with pytest.raises(H.HBGSError) as e:
        g.set_values(to(bad.data))
    assert e.value.code == -4
    for call in (lambda: g.apply(b), lambda: g.apply(b, transpose=True), lambda: g.apply_noalloc(b, out),
                 lambda: g.solve(b), lambda: g.solve(b, transpose=True), lambda: g.get_level(0, 0, "A"),
                 lambda: g.get_level(fields - 1, 0, "AT"), lambda: g.aggregates(0, 0),
                 lambda: g.level_scalars(fields - 1, 0), lambda: g.set_values(to(good.data), rebuild=False)):
        with pytest.raises(H.HBGSError) as e:
            call()
        assert e.value.code == -5
    g.set_values(to(good.data))
    assert torch.equal(g.apply(b), z)
    x, status, _, _ = g.solve(b)
    assert status == 0 and np.allclose(x.cpu().numpy(), np.linspace(1.0, 2.0, n * fields), rtol=1e-7)
