"""The 4-wide collapse on meshes around the size at which its levels go from one workgroup's
loop to launches of their own, with rays that are aimed at triangles and mostly hit: closest
and any hits through both trees are those of a scan over the triangles."""
import numpy as np
import pytest

from .gpu_util import ctx, dev
from .test_gpu_collapse_levels import _mesh

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bvh", ["lbvh", "sah", "ploc"])
@pytest.mark.parametrize("kind,n", [("soup", 2), ("soup", 5), ("soup", 257), ("soup", 4097), ("soup", 13000),
                                    ("chain", 40)])
def test_aimed_rays_hit_what_a_scan_hits(kind, n, bvh):
    import torch
    from paper_2503_12174_amd import dpcs
    mesh = _mesh(kind, n)
    scene = dpcs.Scene(ctx(), mesh, bvh=bvh)
    rng = np.random.default_rng(1)
    m = 1500
    V = mesh.vertices.reshape(n, 3, 3)
    size = np.linalg.norm(V.max(1) - V.min(1), axis=1)

    def check():
        k = rng.choice(np.flatnonzero(size > 1e-2 * size.max()), m)   # (the chain's small ones lie nearer than tmin)
        P = V[k].mean(1)
        N = np.cross(V[k, 1] - V[k, 0], V[k, 2] - V[k, 0]).astype(np.float64)
        N /= np.linalg.norm(N, axis=1, keepdims=True)
        # from within a few sizes of the triangle, near its normal: FP32 origins of far-off
        # triangles would miss the small ones
        d = -N + 0.3 * rng.normal(size=N.shape)
        d /= np.linalg.norm(d, axis=1, keepdims=True)
        o = P - d * (size[k] * rng.uniform(0.5, 3, m))[:, None]
        rays = dev(np.concatenate([o, d, np.full((m, 1), np.inf), np.full((m, 1), -1.0)], 1), torch.float32)
        res = []
        for mode in range(5):
            prim = torch.full((m,), -7, dtype=torch.int32, device="cuda")
            dpcs.dpcs_debug_intersect(ctx(), scene, rays, mode, prim)
            ctx().synchronize()
            res.append(prim.cpu().numpy())
        assert (res[0] >= 0).mean() > 0.9
        for mode in (1, 2):
            np.testing.assert_array_equal(res[mode], res[0], err_msg=f"mode {mode}")
        for mode in (3, 4):
            np.testing.assert_array_equal(res[mode] >= 0, res[0] >= 0, err_msg=f"mode {mode}")
        # rows of origin and direction alone are the same rays
        prim = torch.full((m,), -7, dtype=torch.int32, device="cuda")
        dpcs.dpcs_debug_intersect(ctx(), scene, rays[:, :6].contiguous(), 1, prim)
        ctx().synchronize()
        np.testing.assert_array_equal(prim.cpu().numpy(), res[0])

    check()
    V = (V + 0.05 * size[:, None, None] * rng.normal(size=V.shape) * 0.3).astype(np.float32)
    size = np.linalg.norm(V.max(1) - V.min(1), axis=1)
    scene.refit(dev(V.reshape(-1, 3), torch.float32))
    check()
