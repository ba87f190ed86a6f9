"""The rows of rays handed to the library are the 8 floats per ray that it reads."""
import pytest
import torch

from paper_2503_12174_amd import dpcs


class _Lib:
    """Stands for the library: notes the ray pointer and count of a call."""

    def __init__(self):
        self.calls = []

    def dpcs_debug_intersect(self, ctx, scene, rays, n, *rest):
        self.calls.append((rays, n))
        return dpcs.OK


class _Ctx:
    h = None

    def check(self, st):
        return st

    def synchronize(self):
        pass


@pytest.mark.parametrize("shape", [(5, 7), (5, 3), (5, 9), (40,), (5, 2, 4), (5, 0)])
def test_other_shapes_are_refused(shape, monkeypatch):
    lib = _Lib()
    monkeypatch.setattr(dpcs, "lib", lambda: lib)
    with pytest.raises(ValueError):
        dpcs.dpcs_debug_intersect(_Ctx(), _Ctx(), torch.zeros(shape), 0, torch.zeros(5, dtype=torch.int32))
    assert not lib.calls


@pytest.mark.parametrize("n", [0, 1, 5])
def test_origins_and_directions_get_a_far_end_and_no_triangle_left(n, monkeypatch):
    lib = _Lib()
    monkeypatch.setattr(dpcs, "lib", lambda: lib)
    od = torch.randn(n, 6)
    rows = dpcs.ray_rows(od)
    assert rows.shape == (n, 8) and rows.is_contiguous() and rows.dtype == torch.float32
    assert torch.equal(rows[:, :6], od) and bool((rows[:, 6] == float("inf")).all()) and bool((rows[:, 7] == -1).all())
    prim = torch.zeros(n, dtype=torch.int32)
    dpcs.dpcs_debug_intersect(_Ctx(), _Ctx(), od, 0, prim)
    assert lib.calls[-1][1] == n and lib.calls[-1][0] != od.data_ptr() or n == 0
    full = torch.randn(n, 8)
    dpcs.dpcs_debug_intersect(_Ctx(), _Ctx(), full, 0, prim)
    assert lib.calls[-1] == (full.data_ptr(), n)
