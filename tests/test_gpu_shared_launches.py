"""Independent fields share launches (up to four jobs each): stages whose
fields differ in depth, smoother degree, kernel shape and leaf solver, and
stages of more than four fields, against the oracle.

Bars as for every apply: FP64 <= 1e-13, FP32 V-cycle <= 1e-5 per field;
repeated applies give the same bits.
"""
import numpy as np
import pytest

import oracle
import synth
from parity_util import assert_fields_close

pytestmark = pytest.mark.gpu

SIX = dict(nx=13, ny=11, nz=9, nspecies=3, seed=5)  # 1287 rows per field
OPTS = {
    # one stage of six fields: 4 + 2 jobs per launch; degrees 1 to 4, so that the fields' steps differ
    "six fields, degrees 1-4": dict(block_jacobi=1, coarse_max=60, field_cheb_degree=[1, 2, 3, 4, 2, 1]),
    # V-cycles, Jacobi leaves and (beside them, on their own stream) ILU leaves in one stage
    "mixed leaves": dict(block_jacobi=1, coarse_max=60, field_leaf=[0, 2, 0, 1, 2, 0], ilu_block=100),
    # stages phi_s + p, phi_e, c1 + c2 + c3 with two levels, then one (dense at the finest level)
    "shallow": dict(coarse_max=600),
    "one level": dict(coarse_max=2000),
    # level cap: a dense coarsest level above which every field stops
    "level cap": dict(coarse_max=20, max_levels=2, field_cheb_degree=[2, 4, 2, 2, 3, 2]),
}


@pytest.mark.parametrize("precision,tol", [(0, 1e-13), (1, 1e-5)])
@pytest.mark.parametrize("name", list(OPTS))
def test_stage_apply_parity(name, precision, tol):
    import torch

    import paper_2602_13079_amd as H
    s = synth.make_system(**SIX)
    dev = torch.device("cuda:0")
    opt = OPTS[name]
    g = H.Solver(*(torch.from_numpy(a).to(dev) for a in (s.rowptr, s.col, s.val, s.field_of_row)), s.nf, s.tree,
                 precision=precision, **opt)
    o = oracle.Oracle(s.rowptr, s.col, s.val, s.nf, s.field_of_row, s.tree, precision=precision, **opt)
    r = np.random.default_rng(8).standard_normal(s.n)
    rd = torch.from_numpy(r).to(dev)
    for tr in (False, True):
        z = g.apply(rd, transpose=tr)
        assert_fields_close(z.cpu().numpy(), o.apply(r, transpose=tr), s.field_of_row, tol, (name, tr))
        assert torch.equal(z, g.apply(rd, transpose=tr))
