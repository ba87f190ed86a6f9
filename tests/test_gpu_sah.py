"""The binned SAH build at the edges of its task sizes: a wave's subtree (64 triangles), a
workgroup's chunk (1024) and tasks of several chunks."""
import numpy as np
import pytest

from paper_2503_12174_amd import synth

from .gpu_util import ctx, dev

pytestmark = pytest.mark.gpu


def _soup(n, kind):
    rng = np.random.default_rng(n)
    c = rng.uniform(-1, 1, (n, 1, 3))
    if kind == "line":       # one axis only has extent
        c[:, :, 1:] = 0.25
    elif kind == "copies":   # half of the centroids coincide
        c[n // 2:] = 0.5
    elif kind == "grid":     # equal centroid coordinates, so equal costs and shared bins
        c = np.floor(c * 4) / 4
    v = (c + rng.uniform(-0.1, 0.1, (n, 3, 3)) * rng.uniform(0.1, 1, (n, 1, 1))).astype(np.float32)
    if kind == "copies":
        v[n // 2:] = v[n // 2]
    return synth.Mesh(v.reshape(-1, 3), np.arange(3 * n, dtype=np.int32).reshape(n, 3), np.zeros((n, 3, 2), np.float32))


def _trace(sc, rays, mode):
    import torch
    from paper_2503_12174_amd import dpcs
    n = rays.shape[0]
    prim = torch.zeros(n, dtype=torch.int32, device="cuda")
    t, b1, b2 = (torch.zeros(n, device="cuda") for _ in range(3))
    dpcs.dpcs_debug_intersect(ctx(), sc, rays, mode, prim, t, b1, b2)
    ctx().synchronize()
    return [x.cpu().numpy() for x in (prim, t, b1, b2)]


@pytest.mark.parametrize("kind", ["random", "line", "copies", "grid"])
@pytest.mark.parametrize("n", [1, 2, 3, 33, 63, 64, 65, 66, 128, 1023, 1024, 1025, 1089, 2048, 2113, 9000])
def test_sah_tree_answers_like_brute_force(n, kind):
    """Both trees answer every ray as a scan over the triangles does, bit for bit, and a
    second build of the mesh is the same tree."""
    from paper_2503_12174_amd import dpcs
    mesh = _soup(n, kind)
    sc = dpcs.Scene(ctx(), mesh, bvh="sah")
    a = sc.info()
    rng = np.random.default_rng(7)
    m = 4000
    o = rng.uniform(-2, 2, (m, 3))
    tgt = mesh.vertices.reshape(n, 3, 3)[rng.integers(0, n, m)].mean(1) + rng.normal(0, 0.02, (m, 3))
    d = tgt - o
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    rays = dev(np.concatenate([o, d, np.full((m, 1), np.inf), np.full((m, 1), -1.0)], 1).astype(np.float32))
    ref = _trace(sc, rays, 0)
    assert (ref[0] >= 0).any()
    for mode in (1, 2):
        for x, y in zip(_trace(sc, rays, mode), ref):
            np.testing.assert_array_equal(x, y)
    b = dpcs.Scene(ctx(), mesh, bvh="sah").info()
    assert (a.wide_nodes, a.max_depth, a.num_nodes) == (b.wide_nodes, b.max_depth, b.num_nodes)
    assert a.max_depth <= 64
