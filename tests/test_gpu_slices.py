"""Diagonal slices against the row-block kernels that gather their operand.

The slices replace row blocks of 256 to 32 rows, whose row sums take 1 to 8
partial sums, so each grid below gives one of those counts (rows of a field's
finest level: 262,144 / 257,481 / 82,943 / 36,859); the six-field grid's
transposed outer operator has more than 16 diagonals per slice (32-bit
masks).  Both forms round the products and add them in the same order, so the
results are bitwise the same, and the slices' absent places touch neither
out-of-range nor non-finite operand entries.
"""
import numpy as np
import pytest

import synth
from parity_util import assert_fields_close

pytestmark = pytest.mark.gpu

GRIDS = {
    "1 partial sum": dict(nx=64, ny=64, nz=64),
    "2 partial sums, ragged": dict(nx=67, ny=61, nz=63),
    "4 partial sums, 2D": dict(nx=337, ny=269),
    "8 partial sums, 6 fields": dict(nx=41, ny=29, nz=31, nspecies=3),
}


def _solver(s, precision, **opt):
    import torch

    import paper_2602_13079_amd as H
    dev = torch.device("cuda:0")
    return H.Solver(*(torch.from_numpy(a).to(dev) for a in (s.rowptr, s.col, s.val, s.field_of_row)), s.nf, s.tree,
                    precision=precision, **opt)


def _bits(t):
    a = t.cpu().numpy()
    return np.where(np.isnan(a), np.nan, a).view(np.int64)  # one pattern for every NaN


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("grid", list(GRIDS))
def test_slices_bitwise(grid, precision):
    import torch

    import paper_2602_13079_amd as H
    s = synth.make_system(seed=11, with_dj0=False, **GRIDS[grid])
    g = _solver(s, precision, max_iters=4, rtol=0.0)
    r = torch.from_numpy(np.random.default_rng(3).standard_normal(s.n)).cuda()
    bad = r.clone()
    bad[s.n // 2] = float("inf")  # reaches its neighbours' rows only through entries that exist
    b = torch.from_numpy(s.b).cuda()
    out = {}
    try:
        for on in (True, False):
            H.debug_spmv_tiles(on)
            out[on] = [_bits(g.apply(v, transpose=tr)) for v in (r, bad) for tr in (False, True)]
            for tr in (False, True):
                x, _, _, hist = g.solve(b, transpose=tr)
                out[on] += [_bits(x), np.asarray(hist).view(np.int64)]
    finally:
        H.debug_spmv_tiles(True)
    for k, (p, q) in enumerate(zip(out[True], out[False])):
        assert np.array_equal(p, q), k


@pytest.mark.parametrize("precision,tol", [(0, 1e-13), (1, 1e-5)])
def test_slices_apply_parity(precision, tol):
    """Against the oracle, where the eight-partial-sum form is taken."""
    import torch

    import oracle
    s = synth.make_system(seed=11, with_dj0=False, **GRIDS["8 partial sums, 6 fields"])
    g = _solver(s, precision)
    o = oracle.Oracle(s.rowptr, s.col, s.val, s.nf, s.field_of_row, s.tree, precision=precision)
    r = np.random.default_rng(4).standard_normal(s.n)
    for tr in (False, True):
        z = g.apply(torch.from_numpy(r).cuda(), transpose=tr).cpu().numpy()
        assert_fields_close(z, o.apply(r, transpose=tr), s.field_of_row, tol, tr)
