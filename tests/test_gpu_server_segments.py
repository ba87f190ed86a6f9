"""More requests in a wave than one launch's list of segments holds: every request's pixels
are finalized, differentiated and handed over by its own workgroups."""
import time

import numpy as np
import pytest

from paper_2503_12174_amd import synth

from .gpu_util import ctx, dev
from .test_gpu_server import _setup, _wait

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_req", [2, 16, 17, 35])
def test_wave_of_many_segments(n_req):
    import torch
    from paper_2503_12174_amd import dpcs
    scenes, albedo, rough, spec = _setup(1)
    rng = np.random.default_rng(n_req)
    srv = dpcs.Server(ctx(), budget_bytes=8 << 30, max_slots=40)
    big = synth.corner_50k(spp=64, max_depth=4, res=512, n_quads=20)   # keeps the loop busy while the others queue up
    pb = dpcs.params_from(big, albedo, rough, spec)
    ib, ob = dev(big.proj_image, torch.float32), torch.zeros((512, 512, 3), device="cuda")
    reqs = []
    for k in range(n_req):   # sizes from less than a workgroup of any of the launches to several
        w = synth.corner_50k(spp=(1, 3, 16, 7)[k % 4], max_depth=1 + k % 3, res=(1, 5, 17, 32, 9)[k % 5], n_quads=8)
        pw, ph = 3 + 5 * (k % 7), 11
        w.projector = synth.pinhole((0.85, 0.15, 0.85), (0.3, 0.0, 0.3), 45.0, pw, ph)
        w.seed = k
        p = dpcs.params_from(w, albedo, rough, spec)
        ip = dev(rng.uniform(0, 1, (ph, pw, 3)).astype(np.float32), torch.float32)
        h, wd = w.camera.height, w.camera.width
        out = torch.zeros((h, wd, 3), device="cuda")
        target = grads = None
        if k % 3 != 1:
            target = dev(synth.blob_image(h, wd, 90 + k, lo=0.1, hi=0.9), torch.float32)
            grads = dict(d_proj_image=torch.zeros_like(ip), d_albedo=torch.zeros_like(albedo),
                         d_scalars=torch.zeros(18, device="cuda"))
            if k % 2:
                grads.update(d_roughness=torch.zeros_like(rough), d_specular=torch.zeros_like(spec))
        reqs.append((w, p, ip, out, target, grads))
    torch.cuda.synchronize()
    assert srv.submit(100, scenes[0], pb, ib, ob) == dpcs.OK
    time.sleep(0.002)
    for k, (w, p, ip, out, target, grads) in enumerate(reqs):
        kw = {} if grads is None else dict(target=target, grads=grads)
        assert srv.submit(k, scenes[0], p, ip, out, **kw) == dpcs.OK
    done = _wait(srv, n_req + 1)
    assert sorted(d[0] for d in done) == list(range(n_req)) + [100] and all(d[1] == dpcs.OK for d in done)
    srv.close()
    for k, (w, p, ip, out, target, grads) in enumerate(reqs):
        h, wd = w.camera.height, w.camera.width
        L = torch.zeros((h, wd, w.spp, 3), device="cuda")
        alone = torch.zeros_like(out)
        dpcs.dpcs_render(ctx(), scenes[0], p, ip, alone, sample_radiance=L)
        ctx().synchronize()
        np.testing.assert_array_equal(out.cpu().numpy(), alone.cpu().numpy(), err_msg=f"request {k}")
        if grads is None:
            continue
        G = 2.0 * (alone - target) / (3 * h * wd)
        g2 = {name: torch.zeros_like(v) for name, v in grads.items()}
        dpcs.dpcs_render_vjp(ctx(), scenes[0], p, ip, G.contiguous(), sample_radiance=L, **g2)
        ctx().synchronize()
        for name in grads:   # float sums of at most 2^14 terms in another order
            a, b = grads[name].cpu().numpy(), g2[name].cpu().numpy()
            np.testing.assert_allclose(a, b, rtol=1e-4, atol=1e-5 * (np.abs(b).max() + 1e-30), err_msg=f"{k} {name}")
