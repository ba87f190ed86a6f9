"""Requests that are known to share a wave: a first request waits for its input stream, on
which a kernel spins for a while, and the others are submitted meanwhile.  The loop's counters
say which way they went, their results are those of the plain calls."""
import numpy as np
import pytest

from paper_2503_12174_amd import synth

from .gpu_util import ctx, dev
from .test_gpu_server import _setup, _wait

pytestmark = pytest.mark.gpu


def _request(k, shapes, albedo, rough, spec, rng, depths):
    import torch
    from paper_2503_12174_amd import dpcs
    res, spp = shapes[k % len(shapes)]
    w = synth.corner_50k(spp=spp, max_depth=1 + k % depths, res=res, n_quads=8)
    w.projector = synth.pinhole((0.85, 0.15, 0.85), (0.3, 0.0, 0.3), 45.0, 40 + 3 * k, 31)
    w.seed = k
    ip = dev(rng.uniform(0, 1, (31, 40 + 3 * k, 3)).astype(np.float32), torch.float32)
    grads = dict(d_proj_image=torch.zeros_like(ip), d_albedo=torch.zeros_like(albedo),
                 d_roughness=torch.zeros_like(rough), d_specular=torch.zeros_like(spec),
                 d_scalars=torch.zeros(18, device="cuda"))
    return (w, dpcs.params_from(w, albedo, rough, spec), ip, torch.zeros((res, res, 3), device="cuda"),
            dev(synth.blob_image(res, res, 90 + k, lo=0.1, hi=0.9), torch.float32), grads)


def _spin(ms):
    """Cycles for which torch's spinning kernel takes about ms on this device."""
    import torch
    a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    torch.cuda._sleep(1000)
    a.record()
    torch.cuda._sleep(1 << 20)
    b.record()
    torch.cuda.synchronize()
    return int((1 << 20) * ms / max(a.elapsed_time(b), 0.01))


SMALL = ((64, 32), (33, 9), (100, 3), (51, 19))     # up to 2^17 paths, more than 2^13 on average
LARGE = ((64, 33), (128, 8))                        # 2^17 paths and more: binned one by one
TINY = ((5, 7), (1, 3), (17, 4))                    # below 2^13 on average: one replay by atomics


@pytest.mark.parametrize("shapes,n_req,lists,apart", [(SMALL, 2, 1, 0), (SMALL, 8, 1, 0), (SMALL, 9, 2, 0),
                                                      (SMALL, 17, 3, 0), (LARGE, 3, 0, 3), (TINY, 18, 0, 0)])
def test_requests_that_share_a_wave(shapes, n_req, lists, apart):
    import torch
    from paper_2503_12174_amd import dpcs
    scenes, albedo, rough, spec = _setup(1)
    rng = np.random.default_rng(n_req)
    srv = dpcs.Server(ctx(), budget_bytes=8 << 30, max_slots=24)
    reqs = [_request(k, shapes, albedo, rough, spec, rng, 4) for k in range(n_req)]
    first = synth.corner_50k(spp=1, max_depth=1, res=8, n_quads=8)
    pf, fo = dpcs.params_from(first, albedo, rough, spec), torch.zeros((8, 8, 3), device="cuda")
    fi = dev(first.proj_image, torch.float32)
    cycles = _spin(200.0)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        torch.cuda._sleep(cycles)
    assert srv.submit(100, scenes[0], pf, fi, fo, stream=side) == dpcs.OK
    while (st := srv.stats())["active"] == 0 and st["completed"] == 0:   # until the loop has taken it
        pass
    for k, (w, p, ip, out, target, grads) in enumerate(reqs):
        assert srv.submit(k, scenes[0], p, ip, out, target=target, grads=grads) == dpcs.OK
    done = _wait(srv, n_req + 1)
    assert sorted(d[0] for d in done) == list(range(n_req)) + [100] and all(d[1] == dpcs.OK for d in done)
    waves, st = srv.wave_stats(), srv.stats()
    assert st["waves"] == 2 and waves["most_requests"] == n_req
    assert waves["joint_lists"] == waves["most_lists"] == lists and waves["binned_apart"] == apart
    assert st["replayed_waves"] == 1 and st["binned_waves"] == (1 if lists or apart else 0)
    srv.close()
    for k, (w, p, ip, out, target, grads) in enumerate(reqs):
        h = w.camera.height
        L, alone = torch.zeros((h, h, w.spp, 3), device="cuda"), torch.zeros_like(out)
        dpcs.dpcs_render(ctx(), scenes[0], p, ip, alone, sample_radiance=L)
        ctx().synchronize()
        np.testing.assert_array_equal(out.cpu().numpy(), alone.cpu().numpy(), err_msg=f"request {k}")
        G = 2.0 * (alone - target) / (3 * h * h)
        g2 = {name: torch.zeros_like(v) for name, v in grads.items()}
        dpcs.dpcs_render_vjp(ctx(), scenes[0], p, ip, G.contiguous(), sample_radiance=L, **g2)
        ctx().synchronize()
        for name in grads:   # (G is formed in another order; so are the sums of the scalars)
            a, b = grads[name].cpu().numpy(), g2[name].cpu().numpy()
            np.testing.assert_allclose(a, b, rtol=1e-4, atol=1e-5 * (np.abs(b).max() + 1e-30), err_msg=f"{k} {name}")
