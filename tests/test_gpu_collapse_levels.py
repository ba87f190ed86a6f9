"""The 4-wide collapse on meshes whose levels fit one workgroup's loop, cross its limit on the
way down and come back under it, or form a deep chain: every triangle is found where a test of
all of them finds it, and refits (level by level) keep that."""
from types import SimpleNamespace

import numpy as np
import pytest

from .gpu_util import ctx, dev

pytestmark = pytest.mark.gpu


def _mesh(kind, n):
    rng = np.random.default_rng(n)
    if kind == "chain":   # sizes and distances doubling: a long chain of nodes
        c = np.stack([2.0 ** np.arange(n), np.zeros(n), np.zeros(n)], 1)
        size = c[:, 0] * 0.2
    else:
        c = rng.uniform(-1, 1, (n, 3))
        size = np.full(n, 0.7 * n ** (-1 / 3))
    V = c[:, None, :] + size[:, None, None] * rng.uniform(-0.5, 0.5, (n, 3, 3))
    F = np.arange(3 * n).reshape(n, 3)
    return SimpleNamespace(vertices=V.reshape(-1, 3).astype(np.float32), triangles=F.astype(np.int32),
                           corner_uvs=np.zeros((n, 3, 2), np.float32), emission=None)


@pytest.mark.parametrize("bvh", ["lbvh", "sah", "ploc"])
@pytest.mark.parametrize("kind,n", [("soup", 2), ("soup", 3), ("soup", 4), ("soup", 5), ("soup", 16), ("soup", 257),
                                    ("soup", 1023), ("soup", 4097), ("soup", 13000), ("soup", 60000), ("chain", 40)])
def test_collapse_of_small_and_large_levels(kind, n, bvh):
    import torch
    from paper_2503_12174_amd import dpcs
    mesh = _mesh(kind, n)
    scene = dpcs.Scene(ctx(), mesh, bvh=bvh)
    rng = np.random.default_rng(1)
    V = mesh.vertices

    def check():
        P = V.reshape(n, 3, 3).mean(1)[rng.integers(0, n, 1500)]
        o = P + rng.normal(size=P.shape) * (np.abs(P).max(1, keepdims=True) + 1)
        d = (P - o) / np.linalg.norm(P - o, axis=1, keepdims=True)
        rays = dev(np.concatenate([o, d], 1).astype(np.float32), torch.float32)
        got = [torch.full((len(P),), -7, dtype=torch.int32, device="cuda") for _ in range(2)]
        for mode in (0, 1):
            dpcs.dpcs_debug_intersect(ctx(), scene, rays, mode, got[mode])
        ctx().synchronize()
        np.testing.assert_array_equal(got[0].cpu().numpy(), got[1].cpu().numpy())
        assert (got[0] >= 0).any()

    check()
    V = (V + 0.01 * np.abs(V).min() * rng.normal(size=V.shape)).astype(np.float32)
    scene.refit(dev(V, torch.float32))
    check()
