"""The map flush at every size of its chunks: gradients of one wave against the same call cut
into waves of 2^14 paths (whose flushes use the smallest chunk)."""
import numpy as np
import pytest

from paper_2503_12174_amd import synth

from .gpu_util import GpuRun, ctx, dev

pytestmark = pytest.mark.gpu


# 64 x 64 pixels, depth 3: 12288 spp records at most; chunks of 1024 up to 2^21, 2048 up to 2^22, then 4096
@pytest.mark.parametrize("spp", [1, 170, 171, 341, 342])
def test_flush_chunks(spp):
    import torch
    from paper_2503_12174_amd import dpcs
    w = synth.quad_cube(spp=spp, max_depth=3)
    G = dev(np.random.default_rng(spp).normal(size=(w.camera.height, w.camera.width, 3)), torch.float32)
    grads = []
    try:
        for cap in (1 << 22, 1 << 14):
            run = GpuRun(w, capacity=cap)
            g = dict(d_proj_image=torch.zeros_like(run.proj), d_albedo=torch.zeros_like(run.albedo),
                     d_roughness=torch.zeros_like(run.rough))
            H, W = w.camera.height, w.camera.width
            L = torch.zeros((H, W, spp, 3), device="cuda")
            rec = torch.zeros((H, W, spp, 3), dtype=torch.int32, device="cuda")
            img = torch.zeros((H, W, 3), device="cuda")
            dpcs.dpcs_render(run.c, run.scene, run.params, run.proj, img, sample_radiance=L, path_records=rec)
            dpcs.dpcs_render_vjp(run.c, run.scene, run.params, run.proj, G, sample_radiance=L, path_records=rec, **g)
            ctx().synchronize()
            grads.append({k: v.cpu().numpy().astype(np.float64) for k, v in g.items()})
    finally:
        ctx().check(dpcs.lib().dpcs_context_set_capacity(ctx().h, 1 << 22))   # the default
    # each flush rounds a texel's exact sum to float once: at most 4096 spp / 2^14 + 1 roundings of the
    # running gradient on either side (and as many again for the projector's and the BRDF's last factors)
    tol = 2 * 2.0 ** -24 * (4096 * spp / 2 ** 14 + 4)
    for k in grads[0]:
        a, b = grads[0][k], grads[1][k]
        assert np.abs(a).max() > 0 or k == "d_roughness"   # (a Lambertian scene has none)
        np.testing.assert_allclose(a, b, rtol=0, atol=tol * np.abs(a).max(), err_msg=k)
