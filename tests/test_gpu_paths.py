"""Small waves run whole paths per thread, larger ones (and profiled calls) through the queues:
the same bits in every output."""
import numpy as np
import pytest

from paper_2503_12174_amd import synth

from .gpu_util import GpuRun, ctx

pytestmark = pytest.mark.gpu


def _one_triangle():
    V = np.array([[-0.6, -0.6, 0.0], [0.9, -0.5, 0.02], [0.0, 0.8, -0.01]], np.float32)
    return synth.Mesh(V, np.array([[0, 1, 2]], np.int32), np.random.default_rng(0).uniform(0, 1, (1, 3, 2)).astype(np.float32))


def _case(name):
    if name == "one triangle":   # (no 4-wide tree)
        w = synth.quad_cube(spp=3, max_depth=2)
        w.mesh = _one_triangle()
    elif name == "quad and cube":
        w = synth.quad_cube(spp=4, max_depth=3)
    elif name == "one depth":
        w = synth.quad_cube(spp=1, max_depth=1)
    elif name == "emission":
        w = synth.quad_cube(spp=2, max_depth=5)
        w.mesh = synth.closed_box(0.5)
    else:
        w = synth.corner_50k(spp=5, max_depth=6, res=61, n_quads=40)
        w.env = np.full(3, 0.0 if name == "corner" else 0.04)
        if name == "principled, lit":
            rng = np.random.default_rng(5)
            w.metallic = rng.uniform(0, 1, (512, 512)).astype(np.float32)
            n = rng.uniform(0.4, 0.6, (512, 512, 3))
            n[..., 2] = 1.0
            w.normal_map = n.astype(np.float32)
    return w


@pytest.mark.parametrize("records", [False, True])
@pytest.mark.parametrize("name", ["one triangle", "quad and cube", "one depth", "emission", "corner", "corner, lit",
                                  "principled, lit"])
def test_whole_paths_equal_the_queues(name, records):
    import torch
    from paper_2503_12174_amd import dpcs
    run = GpuRun(_case(name))
    p = run.params
    H, W, c = p.camera.height, p.camera.width, ctx()
    res = []
    for prof in (0, 1):
        c.set_profiling(prof)
        out, lin = (torch.zeros((H, W, 3), device="cuda") for _ in range(2))
        L = torch.zeros((H, W, p.spp, 3), device="cuda")
        hits = torch.zeros((H, W, p.spp, p.max_depth), dtype=torch.int32, device="cuda")
        rec = torch.zeros((H, W, p.spp, p.max_depth), dtype=torch.int32, device="cuda")
        dpcs.dpcs_render(c, run.scene, p, run.proj, out, linear=lin, sample_radiance=L, hit_prims=hits,
                         **(dict(path_records=rec) if records else {}))
        c.synchronize()
        res.append([t.cpu().numpy() for t in (out, lin, L, hits, rec)])
    c.set_profiling(0)
    for a, b in zip(*res):
        np.testing.assert_array_equal(a, b)
    assert (res[0][3] >= 0).any() and res[0][2].max() > 0
    assert not records or (res[0][4] != 0).any()


@pytest.mark.parametrize("env,depth", [(0.0, 3), (0.04, 5)])
def test_edge_paths_equal_the_queues(env, depth):
    """The silhouette part of the camera-pose gradient traces its rays from a queue."""
    from .gpu_util import run_vjp
    w = synth.corner_50k(spp=3, max_depth=depth, res=48, n_quads=20)
    w.env = np.full(3, env)
    G = np.random.default_rng(3).normal(size=(48, 48, 3))
    res = []
    for prof in (0, 1):
        run = GpuRun(w)
        ctx().set_profiling(prof)
        res.append(run_vjp(run, G, mode="records", camera=True, edge_density=32.0))
    ctx().set_profiling(0)
    assert set(res[0]) == set(res[1])
    for k in res[0]:
        if "cam" in k:
            np.testing.assert_array_equal(res[0][k], res[1][k], err_msg=k)
            assert np.abs(res[0][k]).max() > 0


@pytest.mark.parametrize("maps", [True, False])
@pytest.mark.parametrize("name,depth", [("quad and cube", 3), ("corner", 1), ("corner, lit", 4), ("corner, lit", 5)])
def test_whole_replays_equal_the_queues(name, depth, maps):
    """Small waves of up to four depths are replayed whole, others depth by depth: the map sums
    are exact, so every gradient has the same bits."""
    import torch
    from paper_2503_12174_amd import dpcs
    from .gpu_util import dev
    w = _case(name)
    w.max_depth = depth
    run = GpuRun(w)
    p, c = run.params, ctx()
    H, W = p.camera.height, p.camera.width
    G = dev(np.random.default_rng(4).normal(size=(H, W, 3)), torch.float32)
    res = []
    for prof in (0, 1):
        c.set_profiling(prof)
        L = torch.zeros((H, W, p.spp, 3), device="cuda")
        rec = torch.zeros((H, W, p.spp, p.max_depth), dtype=torch.int32, device="cuda")
        img = torch.zeros((H, W, 3), device="cuda")
        dpcs.dpcs_render(c, run.scene, p, run.proj, img, sample_radiance=L, path_records=rec)
        g = dict(d_proj_image=torch.zeros_like(run.proj), d_scalars=torch.zeros(18, device="cuda"))
        if maps:
            g.update(d_albedo=torch.zeros_like(run.albedo), d_roughness=torch.zeros_like(run.rough),
                     d_specular=torch.zeros_like(run.spec))
        dpcs.dpcs_render_vjp(c, run.scene, p, run.proj, G, sample_radiance=L, path_records=rec, **g)
        c.synchronize()
        res.append({k: v.cpu().numpy() for k, v in g.items()})
    c.set_profiling(0)
    for k in res[0]:
        np.testing.assert_array_equal(res[0][k], res[1][k], err_msg=k)
    assert np.abs(res[0]["d_proj_image"]).max() > 0
