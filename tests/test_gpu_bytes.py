"""GPU: the algorithmic bytes of the outer product are those of the form its
matrix is held in, recomputed here from the pattern: diagonal slices (no column
indices, no row pointers), or row blocks with packed columns; and the sum of a
sweep's kernels is the figure for a whole application."""
import numpy as np
import pytest
import scipy.sparse as sp

import synth

pytestmark = pytest.mark.gpu


def _pair(**kw):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_13079_amd as H
    s = synth.make_system(seed=3, with_dj0=False, **kw)
    rp, ci, v, fl = (torch.from_numpy(a).to("cuda:0") for a in (s.rowptr, s.col, s.val, s.field_of_row))
    return torch, s, H.Solver(rp, ci, v, fl, s.nf, s.tree, precision=1)


def _by_field(s):
    """The pattern with the rows and columns of each field together, in the tree's order."""
    order = [f for f in s.tree if f >= 0]
    perm = np.concatenate([np.flatnonzero(s.field_of_row == f) for f in order])
    A = sp.csr_matrix((np.ones(s.nnz), s.col, s.rowptr), shape=(s.n, s.n))[perm][:, perm].tocsr()
    A.sort_indices()
    return A


@pytest.mark.parametrize("kw,mask", [(dict(nx=64, ny=64, nz=64), 2), (dict(nx=41, ny=29, nz=31, nspecies=3), 2),
                                     (dict(nx=337, ny=269), 2)])
def test_slices(kw, mask):
    _, s, g = _pair(**kw)
    A = _by_field(s)
    slices = -(-s.n // 64)
    row = np.repeat(np.arange(s.n), np.diff(A.indptr))
    key = np.unique((row // 64) * (2 * s.n) + (A.indices - row) + s.n)  # (slice, diagonal)
    assert np.bincount(key // (2 * s.n)).max() <= 16 and 64 * key.size <= 1.25 * s.nnz
    for p, x in ((0, 8), (1, 4)):
        want = 64 * key.size * 8 + mask * s.n + 4 * (2 * slices + key.size) + (x + 8) * s.n
        assert g.stats()["spmv_bytes"][p] == want


def test_packed_rows():
    _, s, g = _pair(nx=32, ny=32)
    for p, x in ((0, 8), (1, 4)):
        assert g.stats()["spmv_bytes"][p] == s.nnz * 10 + 4 * (s.n + 1) + 4 * -(-s.nnz // 256) + (x + 8) * s.n


@pytest.mark.parametrize("kw", [dict(nx=64, ny=64, nz=64), dict(nx=41, ny=29, nz=31, nspecies=3), dict(nx=32, ny=32)])
def test_sweep_is_the_sum_of_its_kernels(kw):
    torch, s, g = _pair(**kw)
    b = torch.from_numpy(s.b).cuda()
    g.profile(True)
    iters = g.solve(b)[2]
    t = g.kernel_times()
    g.profile(False)
    parts = sum(v["bytes"] for k, v in t.items() if k.split("_")[0] in ("cheb", "resid", "restrict", "prolong", "coarse",
                                                                        "couple") and k != "spmv_resid")
    assert t["sweep"]["launches"] == iters and t["sweep"]["bytes"] == iters * g.stats()["vcycle_bytes"][1]
    assert abs(parts - t["sweep"]["bytes"]) <= 1e-12 * parts
