"""GPU: ILU leaves on a stream of their own, waited for by the first stage that
reads them or at the sweep's end: in the first, a middle and the last stage,
several at once and in stages after one another, against the oracle.

Bars as for every apply: FP64 <= 1e-13, FP32 <= 1e-5 per field; repeated
applies and solves replayed from graphs give the same bits.
"""
import numpy as np
import pytest

import oracle
import synth
from parity_util import assert_fields_close

pytestmark = pytest.mark.gpu

SIX = dict(nx=13, ny=11, nz=9, nspecies=3, seed=5)
# stages forward: phi_s + p, phi_e, the species (each reads phi_s and phi_e); adjoint: the species + p, phi_e, phi_s
LEAVES = [[2, 0, 0, 0, 0, 0], [0, 2, 0, 0, 0, 0], [0, 0, 2, 0, 0, 0], [0, 0, 0, 2, 0, 2], [2, 0, 2, 0, 2, 0],
          [2, 2, 2, 2, 2, 2], [1, 0, 2, 1, 1, 2]]


@pytest.mark.parametrize("leaf", LEAVES, ids=lambda v: "".join(map(str, v)))
@pytest.mark.parametrize("precision,tol", [(0, 1e-13), (1, 1e-5)])
def test_apply_parity(leaf, precision, tol):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_13079_amd as H
    s = synth.make_system(**SIX)
    dev = torch.device("cuda:0")
    opt = dict(coarse_max=60, field_leaf=leaf, ilu_block=100, precision=precision)
    arrays = [torch.from_numpy(a).to(dev) for a in (s.rowptr, s.col, s.val, s.field_of_row)]
    g = H.Solver(*arrays, s.nf, s.tree, **opt)
    o = oracle.Oracle(s.rowptr, s.col, s.val, s.nf, s.field_of_row, s.tree, **opt)
    r = np.random.default_rng(8).standard_normal(s.n)
    rd = torch.from_numpy(r).to(dev)
    for tr in (False, True):
        z = g.apply(rd, transpose=tr)
        assert_fields_close(z.cpu().numpy(), o.apply(r, transpose=tr), s.field_of_row, tol, (leaf, tr))
        for _ in range(5):
            assert torch.equal(z, g.apply(rd, transpose=tr))
    q = H.Solver(*arrays, s.nf, s.tree, use_graphs=1, **opt)
    b = torch.from_numpy(s.b).to(dev)
    for tr in (False, True):
        want = g.solve(b, transpose=tr)
        for _ in range(3):  # the first captures, the others replay
            got = q.solve(b, transpose=tr)
            assert torch.equal(got[0], want[0]) and got[1:3] == want[1:3]
            assert torch.equal(q.apply(rd, transpose=tr), g.apply(rd, transpose=tr))
