"""The record replay stops at a sample's last lit vertex and forms only the gradients asked
for: what it leaves out must be exactly what contributes nothing."""
import numpy as np
import pytest

from paper_2503_12174_amd import synth

from . import scenes
from .gpu_util import GpuRun, ctx, dev, run_vjp

pytestmark = pytest.mark.gpu


def _corner(depth, env, ext):
    w = synth.corner_50k(spp=3, max_depth=depth, res=37, n_quads=20)
    w.env = np.full(3, env)
    if ext:
        rng = np.random.default_rng(5)
        w.metallic = rng.uniform(0, 1, (512, 512)).astype(np.float32)
        n = rng.uniform(0.4, 0.6, (512, 512, 3))
        n[..., 2] = 1.0
        w.normal_map = n.astype(np.float32)
    return w


def _vjp(run, G, fill=0, **want):
    """VJP from caller's records whose buffer was filled with `fill` before the forward."""
    import torch
    from paper_2503_12174_amd import dpcs
    p = run.params
    H, W = p.camera.height, p.camera.width
    L = torch.zeros((H, W, p.spp, 3), device="cuda")
    rec = torch.full((H, W, p.spp, p.max_depth), fill, dtype=torch.int32, device="cuda")
    img = torch.zeros((H, W, 3), device="cuda")
    dpcs.dpcs_render(run.c, run.scene, p, run.proj, img, sample_radiance=L, path_records=rec)
    like = dict(d_proj_image=run.proj, d_albedo=run.albedo, d_roughness=run.rough, d_specular=run.spec,
                d_metallic=run.metal, d_normal_map=run.nmap, d_scalars=torch.zeros(18, device="cuda"))
    out = {k: torch.zeros_like(v) for k, v in like.items() if v is not None and (not want or k in want)}
    dpcs.dpcs_render_vjp(run.c, run.scene, p, run.proj, dev(G, torch.float32), sample_radiance=L, path_records=rec, **out)
    run.c.synchronize()
    return {k: v.cpu().numpy() for k, v in out.items()}


@pytest.mark.parametrize("depth,env,ext", [(1, 0.0, False), (4, 0.0, False), (6, 0.05, False), (6, 0.05, True)])
def test_words_past_a_paths_end_do_not_matter(depth, env, ext):
    """The forward leaves the words after a path's end as they were: whatever they hold, the
    gradients are the same bits."""
    run = GpuRun(_corner(depth, env, ext))
    G = np.random.default_rng(1).normal(size=(37, 37, 3))
    a, b = _vjp(run, G, fill=0), _vjp(run, G, fill=-1)
    for k in a:
        np.testing.assert_array_equal(a[k], b[k], err_msg=k)


@pytest.mark.parametrize("depth,env,ext", [(1, 0.05, False), (4, 0.05, False), (5, 0.0, True)])
def test_gradients_asked_for_alone(depth, env, ext):
    """Each gradient asked for by itself is the one of the full call (the sums are exact)."""
    run = GpuRun(_corner(depth, env, ext))
    G = np.random.default_rng(2).normal(size=(37, 37, 3))
    full = _vjp(run, G)
    for k in full:
        np.testing.assert_array_equal(_vjp(run, G, **{k: True})[k], full[k], err_msg=k)
        assert np.abs(full[k]).max() > 0, k


def test_samples_without_a_cotangent_or_light_give_zero():
    run = GpuRun(_corner(4, 0.0, False))
    G = np.zeros((37, 37, 3))
    for k, v in _vjp(run, G).items():
        assert not v.any(), k
    run = GpuRun(scenes.c3_ggx(spp=2, seed=3, max_depth=3))
    run.params.projector.t[2] = -100.0   # the projector looks away: every vertex unlit
    for k, v in _vjp(run, np.ones((run.params.camera.height, run.params.camera.width, 3))).items():
        assert not v.any(), k


def test_a_nan_cotangent_reaches_every_map_value_its_paths_touch():
    """A NaN in one pixel's cotangent marks the texels and projector pixels its paths read,
    as far as each path goes on, and no other pixel's."""
    run = GpuRun(_corner(4, 0.0, False))
    H = W = 37
    lit = _vjp(run, np.ones((H, W, 3)))
    G = np.zeros((H, W, 3))
    G[20, 18] = np.nan
    got = _vjp(run, G)
    for k in ("d_albedo", "d_roughness", "d_proj_image"):
        n = np.isnan(got[k]).sum()
        assert 0 < n < 0.5 * got[k].size, k
    assert np.isnan(got["d_scalars"]).any() and np.isfinite(lit["d_albedo"]).all()


@pytest.mark.parametrize("mode", ["own", "records"])
def test_replay_agrees_with_retracing(mode):
    """Records (pruned) against the replay that traces every bounce again (not pruned)."""
    w = _corner(5, 0.05, False)
    run = GpuRun(w)
    G = np.random.default_rng(4).normal(size=(37, 37, 3))
    a, b = run_vjp(run, G, mode=mode), run_vjp(run, G, mode="retrace")
    # FP32 state and sums on both sides: a few hundred roundings of 2^-24 along a path of
    # five vertices, over values of one sign per channel at most partly cancelling
    for k in a:
        assert np.linalg.norm(a[k] - b[k]) <= 2e-5 * np.linalg.norm(b[k]), k
