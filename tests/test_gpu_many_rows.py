"""GPU: a matrix of more than 2^26 rows, beyond which one wavefront per row is
more threads than a launch can have: setup, and solves with A and A^T (whose
rows the setup sorts).  The bound is the solver's own, a true relative residual
of 1e-10, plus the rounding of forming it here (below 1e-14)."""
import pytest

pytestmark = pytest.mark.gpu


def test_more_rows_than_wavefronts():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_13079_amd as H
    n = (1 << 26) + 1027
    dev = torch.device("cuda:0")
    # tridiagonal, not symmetric: row i holds l_i (from row 1 on), 4, u_i (but for the last row)
    rowptr = torch.arange(n + 1, device=dev, dtype=torch.int32) * 3 - 1
    rowptr[0], rowptr[n] = 0, 3 * n - 2
    entry = torch.arange(3 * n - 2, device=dev) + 1
    col = (torch.div(entry, 3, rounding_mode="floor") + entry % 3 - 1).to(torch.int32)
    val = torch.full((3 * n - 2,), 4.0, device=dev, dtype=torch.float64)
    noise = torch.rand(n - 1, device=dev, dtype=torch.float64, generator=torch.Generator(dev).manual_seed(1))
    lower, upper = -0.5 - noise, -1.4 + noise
    val[2::3], val[1::3] = lower, upper
    del entry, noise
    g = H.Solver(rowptr, col, val, torch.zeros(n, dtype=torch.int32, device=dev), 1, [-1, 0, -2], field_leaf=[1],
                 restart=8, rtol=1e-10)
    x = torch.rand(n, device=dev, dtype=torch.float64, generator=torch.Generator(dev).manual_seed(2)) + 0.5
    for tr, (lo, up) in ((False, (lower, upper)), (True, (upper, lower))):
        def times(v):
            y = 4.0 * v
            y[1:] += lo * v[:-1]
            y[:-1] += up * v[1:]
            return y
        b = times(x)
        z, status, _, _ = g.solve(b, transpose=tr)
        res = float(torch.linalg.norm(b - times(z)) / torch.linalg.norm(b))
        assert status == 0 and res <= 1e-10 + 1e-14, (tr, status, res)
