"""GPU: new values on a kept pattern.  A context whose values were replaced, at
sizes where they live in diagonal slices, equals a fresh context of the new
values bit for bit: every hierarchy level, applies and solves in both
directions and precisions, for each leaf, the nested and block Jacobi forms and
the deferred transpose.  A 27-point stencil (more entries in 256 rows than the
load stages) is compared with the oracle after an update."""
import numpy as np
import pytest
import scipy.sparse as sp

import oracle
import synth
from parity_util import assert_fields_close

pytestmark = pytest.mark.gpu

CUBE = dict(nx=41, ny=29, nz=31, nspecies=3)  # 36,859 rows per field, six fields
PLANE = dict(nx=337, ny=269)                  # 90,653 rows per field, four fields
TREE2 = [-1, -1, 0, 1, -2, -1, 2, 3, -2, -2]
CASES = {
    "amg": (CUBE, {}),
    "amg 2D, transpose deferred": (PLANE, dict(build_transpose=0)),
    "one build thread": (PLANE, dict(setup_concurrent=0)),
    "ilu": (CUBE, dict(field_leaf=[0, 0, 0, 2, 2, 2])),
    "jacobi and ilu": (PLANE, dict(field_leaf=[0, 0, 1, 2])),
    "block jacobi": (PLANE, dict(block_jacobi=1)),
    "nested": (PLANE, dict(tree=TREE2, nested=1, restart=5, inner_max_iters=12, field_cheb_degree=[4, 4])),
}


def _everything(torch, g, s, b):
    """Every result that depends on the values, as bytes."""
    out = []
    for f in range(s.nf):
        levels = g.stats()["levels"][f]
        for l in range(levels):
            amg = g.opts.field_leaf[f] == 0
            for w in ("A", "AT") if amg and l + 1 == levels else ("A", "P", "R", "AT") if amg else ("A",):
                out += [a.tobytes() for a in g.get_level(f, l, w)[:3]]
            if amg and l + 1 < levels:
                agg, scalars = g.aggregates(f, l)
                out += [agg.tobytes(), repr(scalars).encode()]
    for precision in (0, 1):
        g.set_precision(precision)
        for tr in (False, True):
            out.append(g.apply(b, transpose=tr).cpu().numpy().tobytes())
            x, _, iters, hist = g.solve(b, transpose=tr)
            out += [x.cpu().numpy().tobytes(), hist.tobytes(), bytes([iters])]
    return out


@pytest.mark.parametrize("name", list(CASES))
def test_update_equals_fresh_context(name):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_13079_amd as H
    grid, opt = CASES[name]
    opt = dict(opt)
    s = synth.make_system(seed=21, with_dj0=False, **grid)
    tree = opt.pop("tree", s.tree)
    rp, ci, v, fl = (torch.from_numpy(a).to("cuda:0") for a in (s.rowptr, s.col, s.val, s.field_of_row))
    # other values: rows and columns scaled, the same matrix only in its pattern
    d = 2.0 ** np.random.default_rng(4).uniform(-1, 1, s.n)
    v2 = torch.from_numpy(s.val * np.repeat(d, np.diff(s.rowptr)) * d[s.col]).to("cuda:0")
    b = torch.from_numpy(s.b).to("cuda:0")
    opt.update(max_iters=6, rtol=0.0)
    fresh = H.Solver(rp, ci, v2, fl, s.nf, tree, **opt)
    assert fresh.debug_layout("A")[0] == "slices"
    assert all(fresh.debug_layout("block", f)[0] == "slices" for f in range(s.nf) if fresh.opts.field_leaf[f] == 0)
    want = _everything(torch, fresh, s, b)
    del fresh
    g = H.Solver(rp, ci, v, fl, s.nf, tree, **opt)
    first = _everything(torch, g, s, b)
    g.set_values(v2)
    assert _everything(torch, g, s, b) == want
    g.set_values(v2, rebuild=False)  # the outer operator alone: the same values again
    assert _everything(torch, g, s, b) == want
    g.set_values(v)
    assert _everything(torch, g, s, b) == first != want


def _stencil27(m):
    """27-point operator on m^3 cells, not symmetric in value."""
    n = m ** 3
    i = np.arange(n).reshape(m, m, m)
    rng = np.random.default_rng(m)
    rows, cols = [], []
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                here, there = ((slice(max(0, -d), m - max(0, d)) for d in q) for q in ((dz, dy, dx), (-dz, -dy, -dx)))
                if dx or dy or dz:
                    rows.append(i[tuple(here)].ravel())
                    cols.append(i[tuple(there)].ravel())
    r, c = np.concatenate(rows), np.concatenate(cols)
    A = sp.coo_matrix((-0.2 - rng.random(r.size), (r, c)), shape=(n, n)).tocsr()
    A = (A + sp.diags(0.1 - np.asarray(A.sum(axis=1)).ravel())).tocsr()
    A.sort_indices()
    return A


@pytest.mark.parametrize("precision,tol", [(0, 1e-13), (1, 1e-5)])
def test_blocks_beyond_the_staging(precision, tol):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_13079_amd as H
    A = _stencil27(33)
    n = A.shape[0]
    assert np.diff(A.indptr[::256]).max() > 4096
    field = np.zeros(n, np.int32)
    opt = dict(theta=[0.0], precision=precision)
    rp, ci, fl = (torch.from_numpy(a).to("cuda:0") for a in (A.indptr.astype(np.int32), A.indices.astype(np.int32), field))
    g = H.Solver(rp, ci, torch.from_numpy(A.data).to("cuda:0"), fl, 1, [-1, 0, -2], **opt)
    assert g.debug_layout("A")[0] == "slices" and g.debug_layout("A")[2] == 32
    assert g.debug_layout("block", 0, precision)[0] == "slices"
    B = A.copy()
    B.data *= np.random.default_rng(1).uniform(0.9, 1.1, B.nnz)
    g.set_values(torch.from_numpy(B.data).to("cuda:0"))
    o = oracle.Oracle(B.indptr.astype(np.int32), B.indices.astype(np.int32), B.data, 1, field, [-1, 0, -2], **opt)
    r = np.random.default_rng(2).standard_normal(n)
    for tr in (False, True):
        z = g.apply(torch.from_numpy(r).cuda(), transpose=tr).cpu().numpy()
        assert_fields_close(z, o.apply(r, transpose=tr), field, tol, tr)
        x, status, _, _ = g.solve(torch.from_numpy(r).cuda(), transpose=tr)
        M = B.T if tr else B
        assert status == 0 and np.linalg.norm(r - M @ x.cpu().numpy()) <= (1e-8 + 1e-13) * np.linalg.norm(r)
