"""GPU: the form each matrix is read in, against the rules restated here from
the pattern.  Slices are taken where 64 consecutive rows keep to at most 32
diagonals, their places are at most 1.25 times the entries, and the row-block
form that they replace has at least 32 rows in a block; masks have 16 bits up
to 16 diagonals.  The grids are those of the bitwise comparison of slices with
row blocks, which would pass without a slice kernel too."""
import numpy as np
import pytest
import scipy.sparse as sp

import synth

pytestmark = pytest.mark.gpu

# grid: rows per block that its finest blocks' slices reproduce
GRIDS = {256: dict(nx=64, ny=64, nz=64), 128: dict(nx=67, ny=61, nz=63), 64: dict(nx=337, ny=269),
         32: dict(nx=41, ny=29, nz=31, nspecies=3)}


def _rows_per_block(M, cap):
    n, found = M.shape[0], 0
    for r in (256, 128, 64, 32, 16, 8, 4):
        ends = M.indptr[np.minimum(np.arange(0, n + r, r), n)]
        most = int(np.diff(ends).max())
        if most == 0 or most > cap:
            continue
        found = r
        if -(-n // r) >= 1024:
            break
    return found


def _form(M, layout_cap, cap):
    """(is it slices, rows per block, mask bits, diagonals)"""
    n, m = M.shape
    row = np.repeat(np.arange(n), np.diff(M.indptr))
    key = np.unique((row // 64) * (n + m) + M.indices - row + n)
    most = int(np.bincount(key // (n + m)).max()) if key.size else 0
    ok = (0 < most <= 32 and 64 * key.size <= 1.25 * M.nnz and _rows_per_block(M, layout_cap) >= 32
          and _rows_per_block(M, 2048) >= 32 and 32 <= _rows_per_block(M, cap) <= 256)
    return (True, _rows_per_block(M, cap), 16 if most <= 16 else 32, most) if ok else (False, 0, 0, 0)


def _csr(M):
    M = M.tocsr()
    M.sort_indices()
    return M


@pytest.mark.parametrize("rb", list(GRIDS))
def test_forms(rb):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_13079_amd as H
    s = synth.make_system(seed=11, with_dj0=False, **GRIDS[rb])
    arrays = (torch.from_numpy(a).to("cuda:0") for a in (s.rowptr, s.col, s.val, s.field_of_row))
    g = H.Solver(*arrays, s.nf, s.tree)
    order = [f for f in s.tree if f >= 0]
    perm = np.concatenate([np.flatnonzero(s.field_of_row == f) for f in order])
    A = _csr(sp.csr_matrix((np.ones(s.nnz), s.col, s.rowptr), shape=(s.n, s.n))[perm][:, perm])
    mats = {("A", 0): A, ("AT", 0): _csr(A.T)}
    lo = 0
    for f in order:
        hi = lo + int((s.field_of_row == f).sum())
        mats["block", f] = _csr(A[lo:hi, lo:hi])
        mats["couplings", f] = _csr(A[lo:hi, :lo]) if lo else None
        mats["couplings_T", f] = _csr(A.T.tocsr()[lo:hi, hi:]) if hi < s.n else None
        lo = hi
    masks = set()
    for (which, f), M in mats.items():
        for precision in (0, 1):
            got = g.debug_layout(which, f, precision)
            if M is None or M.nnz == 0:
                assert got[0] == "none", (which, f, got)
                continue
            # couplings have all the columns before, or behind, the field: their diagonals are column - row all the same
            outer = which in ("A", "AT")
            want = _form(M, 2048 if outer else 4096, 2048 if outer or precision == 0 else 4096)
            assert (got[0] == "slices") == want[0], (which, f, precision, got, want)
            if want[0]:
                assert got[1:] == want[1:], (which, f, precision, got, want)
                masks.add(got[2])
        if which == "block":
            assert got[:2] == ("slices", rb)
    assert masks == ({16, 32} if rb == 32 else {16})


def test_scattered_numbering_is_not_sliced():
    """The same stencil in a random numbering of the cells keeps to no diagonals."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_13079_amd as H
    s = synth.make_system(seed=11, with_dj0=False, nx=64, ny=64, nz=64)
    p = np.random.default_rng(0).permutation(s.n)
    M = _csr(sp.csr_matrix((s.val, s.col, s.rowptr), shape=(s.n, s.n))[p][:, p])
    g = H.Solver(*(torch.from_numpy(a).to("cuda:0") for a in (
        M.indptr.astype(np.int32), M.indices.astype(np.int32), M.data, s.field_of_row[p])), s.nf, s.tree)
    for which, f in [("A", 0), ("AT", 0), ("block", 0), ("couplings", 3)]:
        assert g.debug_layout(which, f)[0] in ("rows", "tiled", "lanes")
    for bad in ((-1, 2, 1), (s.nf, 2, 1), (0, 5, 1), (0, -1, 1), (0, 0, 2)):
        out = (H.ctypes.c_int32 * 4)()
        assert g.lib.hbgs_debug_layout(g.h, *bad, out) == -1
