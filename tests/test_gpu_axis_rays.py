"""Rays that do not move along one or two axes: the 4-wide traversal keeps every triangle a
scan accepts, faces of boxes at the ray's own coordinate included."""
import numpy as np
import pytest

from paper_2503_12174_amd import synth

from .gpu_util import ctx, dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale", [1.0, 1e-3, 1e4])
@pytest.mark.parametrize("name", ["corner", "quad+cube", "closed box"])
def test_axis_parallel_rays_equal_brute_force(name, scale):
    import torch
    from paper_2503_12174_amd import dpcs
    mesh = {"corner": lambda: synth.folded_corner(20, 1, 2), "quad+cube": synth.quad_and_cube,
            "closed box": lambda: synth.closed_box(0.5)}[name]()
    mesh.vertices = (mesh.vertices * np.float32(scale)).astype(np.float32)
    sc = dpcs.Scene(ctx(), mesh, bvh="sah")
    rng = np.random.default_rng(3)
    V = mesh.vertices
    m = 12000
    # origins whose coordinates are vertex coordinates (box faces), 0, or anything
    o = np.stack([V[rng.integers(0, len(V), m), k] for k in range(3)], 1).astype(np.float64)
    o[rng.random((m, 3)) < 0.2] = 0.0
    free = rng.random((m, 3)) < 0.4
    o[free] = (rng.uniform(-0.6, 1.1, (m, 3)) * scale)[free]
    d = rng.normal(size=(m, 3))
    zero = rng.random((m, 3)) < 0.5
    d[zero] = np.where(rng.random(zero.sum()) < 0.3, -0.0, 0.0)
    tiny = (rng.random((m, 3)) < 0.1) & zero
    d[tiny] = rng.choice([1e-30, -1e-30, 1e-40, -1e-42, 1e-20], tiny.sum())
    dead = (np.abs(d) < 1e-10).all(1)
    d[dead, rng.integers(0, 3, dead.sum())] = 1.0
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    rays = dev(np.concatenate([o, d, np.full((m, 1), np.inf), np.full((m, 1), -1.0)], 1).astype(np.float32))
    res = {}
    for mode in (0, 1, 3, 4):
        prim = torch.zeros(m, dtype=torch.int32, device="cuda")
        t, b1, b2 = (torch.zeros(m, device="cuda") for _ in range(3))
        dpcs.dpcs_debug_intersect(ctx(), sc, rays, mode, prim, t, b1, b2)
        ctx().synchronize()
        res[mode] = [x.cpu().numpy() for x in (prim, t, b1, b2)]
    for a, b in zip(res[1], res[0]):
        np.testing.assert_array_equal(a, b)
    np.testing.assert_array_equal(res[3][0] >= 0, res[4][0] >= 0)
    assert (res[0][0] >= 0).mean() > 0.05
