"""Refit level by level: the 4-wide and the binary boxes at every size of level (one
workgroup for several, or a launch of its own), every shape of node, every builder."""
import numpy as np
import pytest

from paper_2503_12174_amd import synth

from .gpu_util import GpuRun, ctx, dev

pytestmark = pytest.mark.gpu


def _soup(n, spacing):
    """n triangles in a row whose distances grow by `spacing` per triangle (a chain of a
    tree when it is 2)."""
    rng = np.random.default_rng(n)
    x = np.cumsum(np.float64(spacing) ** np.arange(n)) if spacing != 1 else np.arange(n)
    x = x / x[-1]
    V = rng.uniform(-0.2, 0.2, (3 * n, 3)) / n
    V[:, 0] += np.repeat(x, 3)
    V[:, 2] += 0.2
    return synth.Mesh(V.astype(np.float32), np.arange(3 * n, dtype=np.int32).reshape(-1, 3),
                      rng.uniform(0, 1, (n, 3, 2)).astype(np.float32))


MESHES = {"2": lambda: _soup(2, 1), "3": lambda: _soup(3, 1), "5": lambda: _soup(5, 1), "chain 48": lambda: _soup(48, 2.0),
          "1000": lambda: _soup(1000, 1), "corner 16k": lambda: synth.folded_corner(63, 5, 6),
          "corner 67k": lambda: synth.folded_corner(129, 5, 6)}


@pytest.mark.parametrize("bvh", ["lbvh", "sah", "ploc"])
@pytest.mark.parametrize("name", list(MESHES))
def test_refit_of_every_level(name, bvh):
    import torch
    from paper_2503_12174_amd import dpcs
    mesh = MESHES[name]()
    sc = dpcs.Scene(ctx(), mesh, bvh=bvh)
    V0 = mesh.vertices
    rng = np.random.default_rng(1)
    ext = (V0.max(0) - V0.min(0)).max()
    V1 = (V0 + rng.normal(size=V0.shape) * 0.01 * ext).astype(np.float32)
    w = synth.quad_cube(spp=2, max_depth=1)
    w.mesh = mesh

    def visits():   # of the camera rays: other queues' order, and with it when a wave tests its leaves, varies
        c = ctx()
        run = GpuRun(w, scene=sc)
        c.set_profiling(2)
        run.render(samples=False, hits=False)
        p = c.profile()
        c.set_profiling(0)
        return p["trace"]["nodes"], p["trace"]["tris"]

    before = visits()
    for V in (V1, V0):
        sc.refit(dev(V, torch.float32))
        m = 2048
        prim = rng.integers(0, len(mesh.triangles), m)
        q = V[mesh.triangles[prim]].astype(np.float64).mean(1)        # aimed at a triangle's middle
        o = q + rng.normal(size=(m, 3)) * ext
        d = q - o
        d /= np.linalg.norm(d, axis=1, keepdims=True)
        rays = dev(np.concatenate([o, d, np.full((m, 1), np.inf), np.full((m, 1), -1.0)], 1).astype(np.float32),
                   torch.float32)
        res = {}
        for mode in range(5):
            prim = torch.zeros(m, dtype=torch.int32, device="cuda")
            t, b1, b2 = (torch.zeros(m, device="cuda") for _ in range(3))
            dpcs.dpcs_debug_intersect(ctx(), sc, rays, mode, prim, t, b1, b2)
            ctx().synchronize()
            res[mode] = [x.cpu().numpy() for x in (prim, t, b1, b2)]
        for mode in (1, 2):
            for a, b in zip(res[mode], res[0]):
                np.testing.assert_array_equal(a, b)
        np.testing.assert_array_equal(res[3][0] >= 0, res[4][0] >= 0)
        assert (res[0][0] >= 0).mean() > 0.5
    assert visits() == before   # back at the first positions: the same boxes, none wider
