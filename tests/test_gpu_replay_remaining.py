"""What remains of a sample's radiance past a vertex is the sample's minus the very
contributions the forward added: with no light beyond the first vertex nothing remains, to the
last bit, however bright that vertex is beside the bounce's reflectance."""
import numpy as np
import pytest

from paper_2503_12174_amd import synth

from .gpu_util import GpuRun, run_vjp

pytestmark = pytest.mark.gpu


def _workload(res, spp, depth):
    """A glossy dark floor whose highlight the camera sees, and a wall that the projector
    reaches with black pixels only: bounces end on a lit vertex of no radiance."""
    q = [[(-1, -1, 0), (1, -1, 0), (1, 1, 0), (-1, 1, 0)], [(1, -1, 0), (1, -1, 2), (1, 1, 2), (1, 1, 0)]]
    V = np.array(q, np.float32).reshape(-1, 3)
    F = np.array([[0, 1, 2], [0, 2, 3], [4, 5, 6], [4, 6, 7]], np.int32)
    c = np.array([(0, 0), (1, 0), (1, 1), (0, 1)])
    uv = np.concatenate([[0.03 + 0.44 * c[:, 0], 0.05 + 0.9 * c[:, 1]], [0.53 + 0.44 * c[:, 0], 0.05 + 0.9 * c[:, 1]]], 1).T
    mesh = synth.Mesh(V, F, uv[F].astype(np.float32))
    cam = synth.pinhole((0.8, 0, 0.8), (0, 0, 0), 30.0, res, res)
    prj = synth.pinhole((-0.8, 0, 0.8), (0.5, 0, 0.1), 70.0, 96, 96)
    # projector pixels whose neighbourhood lies on the floor are bright, the others black
    g = np.arange(-1, 98) + 0.0
    px = np.stack([*np.meshgrid(g, g, indexing="xy"), np.ones((99, 99))], -1)
    d = px @ np.linalg.inv(np.asarray(prj.K).reshape(3, 3)).T @ np.asarray(prj.R).reshape(3, 3)
    o = -np.asarray(prj.R).reshape(3, 3).T @ np.asarray(prj.t)
    hit = o[0] - o[2] * d[..., 0] / np.minimum(d[..., 2], -1e-9)
    floor = (d[..., 2] < 0) & (hit < 0.999)
    on = np.ones((96, 96), bool)
    for dy in range(4):
        for dx in range(4):
            on &= floor[dy:dy + 96, dx:dx + 96]
    img = np.where(on[..., None], np.random.default_rng(1).uniform(0.5, 1, (96, 96, 3)), 0).astype(np.float32)
    t = 64
    rng = np.random.default_rng(2)
    w = synth.Workload("floor and wall", mesh, cam, prj, synth.GGX, rng.uniform(0.005, 0.02, (t, t, 3)).astype(np.float32),
                       np.full((t, t), 0.15, np.float32), np.full((t, t), 1.0, np.float32), img, spp=spp, max_depth=depth,
                       seed=3, clip=False)
    return w


@pytest.mark.parametrize("mode", ["own", "records"])
@pytest.mark.parametrize("ext", [False, True])
@pytest.mark.parametrize("res,spp", [(64, 16), (160, 7)])   # whole replays in one launch, and depth by depth
def test_nothing_remains_past_the_only_light(res, spp, ext, mode):
    maps = dict(metallic=np.full((64, 64), 0.0, np.float32),
                normal_map=np.tile(np.float32([0.5, 0.5, 1.0]), (64, 64, 1))) if ext else {}
    G = np.random.default_rng(5).uniform(0.1, 1, (res, res, 3)).astype(np.float32)
    got = []
    for depth in (1, 2):
        w = _workload(res, spp, depth)
        run = GpuRun(w, **maps)
        got.append(run_vjp(run, G, mode=mode))
        if depth == 2:   # the wall is met and lit
            L = run.render()
            assert (L["hits"][..., 1] >= 2).mean() > 0.1 and (L["L"] > 0).any()
    keys = ["albedo", "roughness", "specular"] + (["metallic", "normal_map"] if ext else [])
    for k in keys:
        one, two = got[0][k], got[1][k]
        assert np.abs(one).max() > 0 or k == "metallic"
        # the same terms, summed exactly and rounded once
        np.testing.assert_allclose(two, one, rtol=2.0 ** -22, atol=2.0 ** -40 * np.abs(one).max(), err_msg=k)
