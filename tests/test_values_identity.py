"""CPU: which value tensors the differentiable solve takes for the ones its
solver holds.  A tensor at the address of a freed one, another stride over the
same storage, an in-place change and a failed update are other values; the
tensor itself and a view of all of it are not.  The library is stubbed: what
counts is when new values are handed to it.
"""
import gc

import pytest
import torch

import paper_2602_13079_amd as H


class _Lib:
    def __init__(self):
        self.loaded, self.code = [], 0

    def hbgs_set_values(self, h, ptr, rebuild, stream):
        self.loaded.append(ptr)
        return self.code

    def hbgs_setup(self, *a):
        return 0

    def hbgs_last_error(self):
        return b"refused"


@pytest.fixture
def held(monkeypatch):
    """[solver that holds `val`, the stub, val]"""
    lib = _Lib()
    monkeypatch.setattr(H, "load", lambda: lib)
    monkeypatch.setattr(H, "_dev", lambda t, dtype, torch: t.contiguous())
    monkeypatch.setattr(H, "_stream", lambda torch: None)
    monkeypatch.setattr(H, "default_options", lambda **kw: H.Options())
    monkeypatch.setattr(H.Solver, "solve", lambda self, b, transpose=False: (b.clone(), 0, 1, None))
    val = torch.full((1000,), 2.0, dtype=torch.float64)
    i = torch.zeros(3, dtype=torch.int32)
    return [H.Solver(i, torch.zeros(val.numel(), dtype=torch.int32), val, i, 1, [-1, 0, -2]), lib, val]


def _solve(solver, val):
    H.hbgs_solve(val, torch.ones(3, dtype=torch.float64), solver)


def test_a_new_tensor_at_a_freed_address_is_loaded(held):
    solver, lib = held[:2]
    for k in range(8):  # a training loop: other values each step, the previous ones freed
        n = len(lib.loaded)
        held[2:] = []
        gc.collect()
        held.append(torch.full((1000,), 3.0 + k, dtype=torch.float64))
        _solve(solver, held[2])
        assert len(lib.loaded) == n + 1, k


def test_the_same_values_are_not_loaded_again(held):
    solver, lib, val = held
    for v in (val, val.detach(), val.view(-1)):
        _solve(solver, v)
    assert lib.loaded == []


def test_changes_are_loaded(held):
    solver, lib, val = held
    val.mul_(2.0)
    _solve(solver, val)
    _solve(solver, val)
    assert len(lib.loaded) == 1
    _solve(solver, val[:1].expand(val.numel()))  # the same address, size and version
    assert len(lib.loaded) == 2


def test_a_failed_update_leaves_no_known_values(held):
    solver, lib, val = held
    lib.code = -4
    with pytest.raises(H.HBGSError):
        solver.set_values(val.clone())
    lib.code = 0
    _solve(solver, val)
    assert len(lib.loaded) == 2
