"""Several compensation requests of one wave: each replays and bins by itself, at its own
place in the wave's samples and records."""
import time

import numpy as np
import pytest

from paper_2503_12174_amd import synth

from .gpu_util import ctx, dev
from .test_gpu_server import _setup, _wait

pytestmark = pytest.mark.gpu


def test_several_requests_of_a_wave_bin_their_gradients():
    import torch
    from paper_2503_12174_amd import dpcs
    scenes, albedo, rough, spec = _setup(1)
    rng = np.random.default_rng(9)
    srv = dpcs.Server(ctx(), budget_bytes=8 << 30, max_slots=16)
    big = synth.corner_50k(spp=64, max_depth=4, res=512, n_quads=20)   # keeps the loop busy while the others queue up
    pb = dpcs.params_from(big, albedo, rough, spec)
    ib, ob = dev(big.proj_image, torch.float32), torch.zeros((512, 512, 3), device="cuda")
    reqs = []
    for k in range(6):   # 2^17 paths each: where several requests of a wave are binned one by one
        res = (64, 128)[k % 2]
        w = synth.corner_50k(spp=(32, 8)[k % 2], max_depth=1 + k % 5, res=res, n_quads=8)
        w.projector = synth.pinhole((0.85, 0.15, 0.85), (0.3, 0.0, 0.3), 45.0, 40 + 16 * k, 48)
        w.seed = k
        img = rng.uniform(0, 1, (48, 40 + 16 * k, 3)).astype(np.float32)
        p = dpcs.params_from(w, albedo, rough, spec)
        ip = dev(img, torch.float32)
        out = torch.zeros((w.camera.height, w.camera.width, 3), device="cuda")
        target = dev(synth.blob_image(w.camera.height, w.camera.width, 90 + k, lo=0.1, hi=0.9), torch.float32)
        grads = dict(d_proj_image=torch.zeros_like(ip), d_albedo=torch.zeros_like(albedo),
                     d_roughness=torch.zeros_like(rough), d_specular=torch.zeros_like(spec),
                     d_scalars=torch.zeros(18, device="cuda"))
        reqs.append((w, p, ip, out, target, grads))
    torch.cuda.synchronize()
    s0 = srv.stats()
    assert srv.submit(100, scenes[0], pb, ib, ob) == dpcs.OK
    time.sleep(0.002)
    for k, (w, p, ip, out, target, grads) in enumerate(reqs):
        assert srv.submit(k, scenes[0], p, ip, out, target=target, grads=grads) == dpcs.OK
    done = _wait(srv, 7)
    assert sorted(d[0] for d in done) == list(range(6)) + [100] and all(d[1] == dpcs.OK for d in done)
    s1 = srv.stats()
    assert s1["binned_waves"] - s0["binned_waves"] == s1["replayed_waves"] - s0["replayed_waves"] > 0
    srv.close()
    for k, (w, p, ip, out, target, grads) in enumerate(reqs):
        L = torch.zeros((w.camera.height, w.camera.width, w.spp, 3), device="cuda")
        alone = torch.zeros_like(out)
        dpcs.dpcs_render(ctx(), scenes[0], p, ip, alone, sample_radiance=L)
        ctx().synchronize()
        np.testing.assert_array_equal(out.cpu().numpy(), alone.cpu().numpy(), err_msg=f"request {k}")
        G = 2.0 * (alone - target) / (3 * w.camera.height * w.camera.width)
        g2 = {name: torch.zeros_like(v) for name, v in grads.items()}
        dpcs.dpcs_render_vjp(ctx(), scenes[0], p, ip, G.contiguous(), sample_radiance=L, **g2)
        ctx().synchronize()
        for name in grads:
            a, b = grads[name].cpu().numpy(), g2[name].cpu().numpy()
            np.testing.assert_allclose(a, b, rtol=1e-4, atol=1e-5 * (np.abs(b).max() + 1e-30), err_msg=f"{k} {name}")


@pytest.mark.parametrize("n_req", [2, 8, 9, 17])
def test_small_requests_of_a_wave_replay_and_flush_together(n_req):
    import torch
    from paper_2503_12174_amd import dpcs
    scenes, albedo, rough, spec = _setup(1)
    rng = np.random.default_rng(n_req)
    srv = dpcs.Server(ctx(), budget_bytes=8 << 30, max_slots=24)
    big = synth.corner_50k(spp=64, max_depth=4, res=512, n_quads=20)   # keeps the loop busy while the others queue up
    pb = dpcs.params_from(big, albedo, rough, spec)
    ib, ob = dev(big.proj_image, torch.float32), torch.zeros((512, 512, 3), device="cuda")
    reqs = []
    for k in range(n_req):   # up to 2^17 paths and 4 depths, 4,096 paths on average or more; maps of other sizes
        res, spp = ((64, 32), (33, 7), (100, 3), (51, 19))[k % 4]
        w = synth.corner_50k(spp=spp, max_depth=1 + k % 4, res=res, n_quads=8)
        pw, ph = (40, 257, 129, 8, 1)[k % 5], (48, 31, 1)[k % 3]
        w.projector = synth.pinhole((0.85, 0.15, 0.85), (0.3, 0.0, 0.3), 45.0, pw, ph)
        w.seed = k
        t = (16, 61, 5)[k % 3]
        maps = [m[:t, :t + k % 2].contiguous() for m in (albedo, rough, spec)]
        p = dpcs.params_from(w, *maps)
        ip = dev(rng.uniform(0, 1, (ph, pw, 3)).astype(np.float32), torch.float32)
        h, wd = w.camera.height, w.camera.width
        out = torch.zeros((h, wd, 3), device="cuda")
        target = dev(synth.blob_image(h, wd, 90 + k, lo=0.1, hi=0.9), torch.float32)
        grads = dict(d_proj_image=torch.zeros_like(ip), d_albedo=torch.zeros_like(maps[0]),
                     d_roughness=torch.zeros_like(maps[1]), d_specular=torch.zeros_like(maps[2]),
                     d_scalars=torch.zeros(18, device="cuda"))
        reqs.append((w, p, ip, out, target, grads, maps))
    torch.cuda.synchronize()
    s0 = srv.stats()
    assert srv.submit(100, scenes[0], pb, ib, ob) == dpcs.OK
    time.sleep(0.002)
    for k, (w, p, ip, out, target, grads, maps) in enumerate(reqs):
        assert srv.submit(k, scenes[0], p, ip, out, target=target, grads=grads) == dpcs.OK
    done = _wait(srv, n_req + 1)
    assert sorted(d[0] for d in done) == list(range(n_req)) + [100] and all(d[1] == dpcs.OK for d in done)
    s1 = srv.stats()
    assert s1["binned_waves"] - s0["binned_waves"] == s1["replayed_waves"] - s0["replayed_waves"] > 0
    srv.close()
    for k, (w, p, ip, out, target, grads, maps) in enumerate(reqs):
        h, wd = w.camera.height, w.camera.width
        L = torch.zeros((h, wd, w.spp, 3), device="cuda")
        alone = torch.zeros_like(out)
        dpcs.dpcs_render(ctx(), scenes[0], p, ip, alone, sample_radiance=L)
        ctx().synchronize()
        np.testing.assert_array_equal(out.cpu().numpy(), alone.cpu().numpy(), err_msg=f"request {k}")
        G = 2.0 * (alone - target) / (3 * h * wd)
        g2 = {name: torch.zeros_like(v) for name, v in grads.items()}
        dpcs.dpcs_render_vjp(ctx(), scenes[0], p, ip, G.contiguous(), sample_radiance=L, **g2)
        ctx().synchronize()
        for name in grads:   # (G is formed in another order; sums of the scalars too)
            a, b = grads[name].cpu().numpy(), g2[name].cpu().numpy()
            np.testing.assert_allclose(a, b, rtol=1e-4, atol=1e-5 * (np.abs(b).max() + 1e-30), err_msg=f"{k} {name}")
