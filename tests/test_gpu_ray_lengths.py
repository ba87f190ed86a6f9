"""Directions need not be unit vectors: the 4-wide traversal answers rays of any direction
length as a scan over the triangles does, axes without movement included."""
import numpy as np
import pytest

from paper_2503_12174_amd import synth

from .gpu_util import ctx, dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("length", [1e-32, 1e-27, 1e-24, 1e-20, 0.01, 1.0, 30.0])
def test_directions_of_any_length(length):
    import torch
    from paper_2503_12174_amd import dpcs
    mesh = synth.folded_corner(20, 1, 2)
    sc = dpcs.Scene(ctx(), mesh, bvh="sah")
    rng = np.random.default_rng(4)
    m = 6000
    d = rng.normal(size=(m, 3))
    d[rng.random((m, 3)) < 0.2] = 0.0
    d[np.abs(d).max(1) == 0, 0] = 1.0
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    P = mesh.vertices[mesh.triangles].mean(1)[rng.integers(0, len(mesh.triangles), m)]
    o = P - 0.3 * d
    rays = dev(np.concatenate([o, d * length, np.full((m, 1), np.inf), np.full((m, 1), -1.0)], 1), torch.float32)
    res = []
    for mode in range(5):
        prim = torch.full((m,), -7, dtype=torch.int32, device="cuda")
        t = torch.zeros(m, device="cuda")
        dpcs.dpcs_debug_intersect(ctx(), sc, rays, mode, prim, t)
        ctx().synchronize()
        res.append((prim.cpu().numpy(), t.cpu().numpy()))
    assert (res[0][0] >= 0).mean() > 0.5
    for mode in (1, 2):
        np.testing.assert_array_equal(res[mode][0], res[0][0], err_msg=f"mode {mode}")
        np.testing.assert_array_equal(res[mode][1], res[0][1], err_msg=f"mode {mode}")
    np.testing.assert_array_equal(res[3][0] >= 0, res[4][0] >= 0)
