"""The work a user of the renderer has it do, through its public entry points: one case per
use, over the sizes of this repository's own workloads (synth.py, bench.py, the tests) and
around them.

A case is a dict of plain values.  `quads` is the resolution of the projection surface:
0 is the quad and cube (14 triangles), n > 0 a folded corner of n x n quads per plane with
three boxes (4 n^2 + 36 triangles).  `cw, ch` is the camera, `pw, ph` the projector, `tex`
the side of the BRDF maps.  Kinds:

  relight     one forward render of a projector image (simulating a projection)
  step        forward keeping per-sample radiance and path records, then the VJP of every
              map, the projector image and the response scalars (scene fitting on the
              C-level entry points); `mode` "own" lets the VJP run its forward itself,
              "retrace" gives it the radiance alone; `ext` adds the metallic and normal maps
  fit         one image pair of a scene fit through torch autograd (L2 loss)
  compensate  one projector-compensation step through torch autograd: only the projector
              image is optimised
  batch       one scene-fit step of several image pairs through the request loop
  pose        the camera-pose gradient (interior and edge parts) with a VJP from records
  objective   the paper's objective on renderings: guide features, the denoiser, the L1 term
              and the regulariser of the three maps, with all gradients
  build       residency of a new surface: upload, tree build, its guide features
  refit       a moving surface: the tree refitted to new vertices, one relit frame
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2503_12174_amd import autograd, dpcs, objective, synth

LAMBERT, GGX = 0, 1


def _case(name, kind, **kw):
    c = dict(kind=kind, quads=112, cw=256, ch=256, pw=256, ph=256, tex=512, spp=16, depth=4, brdf=GGX, env=0.0,
             mode="records", ext=False, pairs=1, bvh="sah", radius=3, density=0.0)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest render: interactive preview of a toy scene, all launch latency
        _case("relight_quad_cube_64", "relight", quads=0, cw=64, ch=64, pw=64, ph=64, tex=64, spp=4, depth=3,
              brdf=LAMBERT, bvh="lbvh"),
        # one pair of the scene fit through autograd (the drivers' per-pair step)
        _case("fit_quad_cube_64", "fit", quads=0, cw=64, ch=64, pw=64, ph=64, tex=64, spp=32, depth=3, bvh="lbvh"),
        # the scene fit's step: eight pairs in the request loop
        _case("batch_fit_8x64", "batch", quads=0, cw=64, ch=64, pw=64, ph=64, tex=64, spp=32, depth=3, pairs=8,
              bvh="lbvh"),
        # relighting at the benchmark's scale, projector alone
        _case("relight_corner50k_256", "relight", spp=64),
        # relighting at the paper's capture sizes, in a lit room
        _case("relight_capture_env", "relight", cw=640, ch=360, pw=800, ph=600, env=0.05),
        # the benchmark's step: forward and VJP of everything
        _case("step_corner50k_256", "step", spp=64),
        # the full principled BRDF on a ragged image, longer paths, lit room
        _case("step_principled_ragged", "step", cw=317, ch=203, pw=300, ph=217, tex=500, spp=9, depth=6, env=0.03,
              ext=True),
        # projector compensation at its own scale (200k triangles, 512^2)
        _case("compensate_corner200k_512", "compensate", quads=224, cw=512, ch=512, pw=512, ph=512),
        # camera-pose refinement: interior and silhouette terms
        _case("pose_corner50k_256", "pose", density=4.0),
        # the paper's objective at its capture size
        _case("objective_640x360", "objective", quads=0, cw=640, ch=360, pw=64, ph=64, bvh="lbvh"),
        # a new 200k-triangle surface
        _case("build_corner200k", "build", quads=224, cw=256, ch=256),
        # a frame of a moving surface
        _case("refit_relight_corner50k", "refit", cw=640, ch=360, pw=800, ph=600, spp=4),
    ]


MAX_PATHS, MAX_VERTICES = 1 << 21, 1 << 23   # half the largest listed render's


def draw(rng):
    def size(lo, hi, odd=True):   # spread over the logarithm, odd sizes among them
        v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
        return v if odd else max(lo, v // 8 * 8)

    kind = rng.choice(["relight", "relight", "step", "step", "fit", "compensate", "batch", "pose", "objective",
                       "build", "refit"])
    toy = kind in ("fit", "batch", "objective") or (kind in ("relight", "step") and rng.random() < 0.4)
    c = _case(None, kind, quads=0 if toy else size(24, 224), bvh=rng.choice(["lbvh", "sah", "ploc"]),
              brdf=GGX if rng.random() < 0.8 else LAMBERT, env=0.0 if rng.random() < 0.5 else round(rng.uniform(0.01, 0.2), 3),
              tex=size(32, 512), pw=size(32, 640), ph=size(32, 512))
    big = 128 if kind == "batch" else 640
    c["cw"], c["ch"] = size(40, big), size(40, big * 3 // 4)
    c["depth"] = rng.randint(1, 8) if rng.random() < 0.4 else rng.choice([3, 4])
    cap = MAX_PATHS if kind not in ("batch", "fit", "pose") else 1 << 20
    c["spp"] = size(1, 64)
    while c["spp"] > 1 and (c["cw"] * c["ch"] * c["spp"] > cap or c["cw"] * c["ch"] * c["spp"] * c["depth"] > MAX_VERTICES):
        c["spp"] = max(1, c["spp"] // 2)
    if kind == "step":
        c["ext"] = rng.random() < 0.25 and c["brdf"] == GGX
        c["mode"] = rng.choice(["records", "records", "own"] + ([] if c["ext"] else ["retrace"]))
    if kind in ("fit", "batch", "compensate", "pose", "objective"):
        c["brdf"] = GGX
    if kind == "batch":
        c["pairs"] = rng.randint(2, 8)
        while c["pairs"] > 2 and c["cw"] * c["ch"] * c["spp"] * c["pairs"] > 1 << 20:
            c["pairs"] -= 1
        while c["spp"] > 1 and c["cw"] * c["ch"] * c["spp"] * c["pairs"] > 1 << 20:
            c["spp"] = max(1, c["spp"] // 2)
    if kind == "pose":
        c["density"] = rng.choice([0.0, 1.0, 4.0])
    if kind == "objective":
        c["radius"] = rng.randint(1, 6)
    return c


# ------------------------------------------------------------------ inputs

_contexts = {}


def _context():
    """The program's one context (it keeps its scratch from call to call)."""
    dev = torch.cuda.current_device()
    if dev not in _contexts:
        _contexts[dev] = dpcs.Context(dev)
    return _contexts[dev]


def _mesh(case, seed):
    if case["quads"] == 0:
        return synth.quad_and_cube()
    return synth.folded_corner(case["quads"], 201 + seed, 202 + seed)


def _workload(case, seed):
    """Host-side workload; the seed moves the surface, maps, images and sample paths."""
    rng = np.random.default_rng([seed, 7])
    t, cw, ch, pw, ph = case["tex"], case["cw"], case["ch"], case["pw"], case["ph"]
    albedo = rng.uniform(0.2, 0.8, (t, t, 3)).astype(np.float32)
    rough = rng.uniform(0.1, 0.9, (t, t)).astype(np.float32)
    spec = rng.uniform(0.0, 1.0, (t, t)).astype(np.float32)
    if case["quads"] == 0:
        ang = math.radians(30.0)
        eye_p = (-0.6 * math.sin(ang), 0.0, 0.6 * math.cos(ang))
        projector = synth.pinhole(eye_p, (0, 0, 0), 60.0, pw, ph, up=(0, 1, 0))
        camera = synth.pinhole((0, 0, 0.8), (0, 0, 0), 60.0, cw, ch, up=(0, 1, 0))
        image = rng.uniform(0, 1, (ph, pw, 3)).astype(np.float32)
    else:
        projector = synth.pinhole((0.85, 0.15, 0.85), (0.3, 0.0, 0.3), 45.0, pw, ph)
        camera = synth.pinhole((0.85, 0.0, 0.85), (0.3, 0.0, 0.3), 60.0, cw, ch)
        image = synth.blob_image(ph, pw, 204 + seed)
    ext = {}
    if case["ext"]:
        n = np.stack([rng.uniform(0.35, 0.65, (t, t)), rng.uniform(0.35, 0.65, (t, t)), rng.uniform(0.9, 1.0, (t, t))], -1)
        ext = dict(metallic=rng.uniform(0, 1, (t, t)).astype(np.float32), normal_map=n.astype(np.float32))
    w = synth.Workload("case", _mesh(case, seed), camera, projector, case["brdf"], albedo, rough, spec, image,
                       white_balance=np.array([1.0, 0.95, 1.05]), env=np.full(3, case["env"]), spp=case["spp"],
                       max_depth=case["depth"], seed=seed & 0xffff, **ext)
    # float32 values throughout, so a 64-bit evaluation starts from the same inputs
    for k in ("prf_gamma", "prf_mix", "crf_gamma", "white_balance", "env"):
        setattr(w, k, np.asarray(getattr(w, k), np.float32).astype(np.float64))
    return w, rng


def _dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, np.float32)).cuda()


def prepare(case, seed):
    w, rng = _workload(case, seed)
    ctx = _context()
    kind = case["kind"]
    s = dict(case=case, ctx=ctx, w=w)
    maps = s["maps"] = [_dev(w.albedo), _dev(w.roughness), _dev(w.specular)]
    s["ext"] = {} if not case["ext"] else dict(metallic=_dev(w.metallic), normal_map=_dev(w.normal_map))
    proj = s["proj"] = _dev(w.proj_image)
    H, W = case["ch"], case["cw"]
    s["params"] = dpcs.params_from(w, *maps, **s["ext"])
    s["out"] = torch.zeros((H, W, 3), device="cuda")
    if kind == "build":
        return s
    s["scene"] = dpcs.Scene(ctx, w.mesh, bvh=case["bvh"])
    if kind == "refit":   # a billowing of the surface, as a user's animation gives it
        V = w.mesh.vertices
        k = 0.01 * np.sin(2 * np.pi * (V @ np.array([2.0, 3.0, 1.0]) + rng.uniform()))
        s["positions"] = _dev(V + k[:, None] * np.array([0.5, 0.2, 0.5]))
    if kind in ("step", "pose"):
        s["G"] = _dev(rng.normal(size=(H, W, 3)))
        if case["mode"] != "own":
            s["L"] = torch.zeros((H, W, w.spp, 3), device="cuda")
        if case["mode"] == "records":
            s["rec"] = torch.zeros((H, W, w.spp, w.max_depth), dtype=torch.int32, device="cuda")
        s["grads"] = dict(d_proj_image=torch.zeros_like(proj), d_albedo=torch.zeros_like(maps[0]),
                          d_roughness=torch.zeros_like(maps[1]), d_specular=torch.zeros_like(maps[2]),
                          d_scalars=torch.zeros(dpcs.NUM_SCALARS, device="cuda"))
        if case["ext"]:
            s["grads"].update(d_metallic=torch.zeros_like(maps[1]), d_normal_map=torch.zeros_like(maps[0]))
        if kind == "pose":
            s["grads"]["d_camera"] = torch.zeros(12, device="cuda")
    if kind in ("fit", "compensate"):
        s["scal"] = autograd.scalars_from(w)
        s["target"] = _dev(rng.uniform(0, 1, (H, W, 3)))
        if kind == "fit":
            for t in maps + [s["scal"]]:
                t.requires_grad_(True)
        else:
            proj.requires_grad_(True)
    if kind == "batch":
        n = case["pairs"]
        s["scal"] = autograd.scalars_from(w)
        s["images"] = [_dev(rng.uniform(0, 1, (case["ph"], case["pw"], 3))) for _ in range(n)]
        s["targets"] = [_dev(rng.uniform(0, 1, (H, W, 3))) for _ in range(n)]
        s["params"] = dpcs.params_from(w, *maps, device_scalars=s["scal"])
        paths = H * W * w.spp * n
        s["server"] = dpcs.Server(ctx, budget_bytes=max(1 << 30, 4 * 640 * paths + (256 << 20)), max_slots=n)
        s["next_id"] = 0
    if kind == "objective":
        s["cfg"] = objective.DenoiseConfig(radius=case["radius"])
        s["image"] = _dev(rng.uniform(0, 1, (H, W, 3))).requires_grad_(True)   # a noisy rendering
        s["target"] = _dev(rng.uniform(0, 1, (H, W, 3)))
        for t in maps:
            t.requires_grad_(True)
    return s


# ------------------------------------------------------------------ one pass

def _relight(s):
    dpcs.dpcs_render(s["ctx"], s["scene"], s["params"], s["proj"], s["out"])
    return s["out"]


def _step(s):
    ctx, sc, p, proj = s["ctx"], s["scene"], s["params"], s["proj"]
    L, rec = s.get("L"), s.get("rec")
    if L is not None:
        dpcs.dpcs_render(ctx, sc, p, proj, s["out"], sample_radiance=L, path_records=rec)
    dpcs.dpcs_render_vjp(ctx, sc, p, proj, s["G"], sample_radiance=L, path_records=rec,
                         camera_edge_density=s["case"]["density"], **s["grads"])
    return dict(image=s["out"], **s["grads"]) if L is not None else dict(s["grads"])


def _autograd(s, leaves):
    a, r, sp = s["maps"]
    out = autograd.render(s["ctx"], s["scene"], s["w"], s["proj"], a, r, sp, s["scal"])
    loss = ((out - s["target"]) ** 2).mean()
    for t in leaves:
        t.grad = None
    loss.backward()
    return dict(image=out.detach(), grads=[t.grad for t in leaves])


def _batch(s):
    srv, a, r, sp = s["server"], *s["maps"]
    outs, grads = [], []
    for ip, tgt in zip(s["images"], s["targets"]):
        out = torch.empty_like(tgt)
        g = dict(d_albedo=torch.zeros_like(a), d_roughness=torch.zeros_like(r), d_specular=torch.zeros_like(sp),
                 d_scalars=torch.zeros_like(s["scal"]))
        st = srv.submit(s["next_id"], s["scene"], s["params"], ip, out, target=tgt, grads=g)
        if st != dpcs.OK:
            raise RuntimeError(f"request refused: status {st}")
        s["next_id"] += 1
        outs.append(out)
        grads.append(g)
    done = 0
    while done < len(outs):
        for _, st, _ in srv.poll():
            if st != dpcs.OK:
                raise RuntimeError(f"request failed: status {st}")
            done += 1
    return dict(images=outs, grads={k: sum(g[k] for g in grads) / len(grads) for k in grads[0]})


def _objective(s):
    ctx, (a, r, sp) = s["ctx"], s["maps"]
    guide = objective.gbuffer(ctx, s["scene"], s["params"])
    loss = objective.l1(ctx, objective.denoise(ctx, s["image"], guide, s["cfg"]), s["target"])
    loss = loss + 0.1 * (objective.tv(ctx, a) + objective.tv(ctx, r) + objective.tv(ctx, sp))
    leaves = [s["image"], a, r, sp]
    for t in leaves:
        t.grad = None
    loss.backward()
    return dict(loss=loss.detach(), guide=guide, grads=[t.grad for t in leaves])


def _build(s):
    scene = dpcs.Scene(s["ctx"], s["w"].mesh, bvh=s["case"]["bvh"])
    guide = objective.gbuffer(s["ctx"], scene, s["params"])
    scene.close()   # (waits for the stream)
    return guide


def run(s):
    kind = s["case"]["kind"]
    if kind == "relight":
        return _relight(s)
    if kind in ("step", "pose"):
        return _step(s)
    if kind == "fit":
        return _autograd(s, s["maps"] + [s["scal"]])
    if kind == "compensate":
        return _autograd(s, [s["proj"]])
    if kind == "batch":
        return _batch(s)
    if kind == "objective":
        return _objective(s)
    if kind == "build":
        return _build(s)
    s["scene"].refit(s["positions"])
    return _relight(s)


# ------------------------------------------------------------------ work

def work(case):
    """Bytes: every input read once, every output written once.  Operations: per ray the
    slabs of a 4-wide tree on a path to its leaf and two triangles; per vertex the surface,
    the lookups and the reflectance (about twice that again in a VJP)."""
    kind, n = case["kind"], case["pairs"]
    tris = 14 if case["quads"] == 0 else 4 * case["quads"] ** 2 + 36
    pix, px, tex = case["cw"] * case["ch"], case["pw"] * case["ph"], case["tex"] ** 2
    channels = 9 if case["ext"] else 5
    mesh, maps = tris * (12 + 24 + 6), 4 * channels * tex
    ray = 58 + 75 * (1 + math.log(max(tris, 4), 4)) + 66
    vertices = pix * case["spp"] * (1 + 0.5 * (case["depth"] - 1))   # about half the bounces stay in the scene
    forward = vertices * (1.5 * ray + 300)
    if kind == "relight":
        return dict(bytes=mesh + maps + 12 * px + 12 * pix, flops=forward)
    if kind == "refit":
        return dict(bytes=2 * mesh + maps + 12 * px + 12 * pix, flops=forward + 100 * tris)
    if kind in ("step", "fit", "pose"):
        return dict(bytes=mesh + 2 * maps + 24 * px + 24 * pix, flops=forward + 600 * vertices)
    if kind == "compensate":
        return dict(bytes=mesh + maps + 24 * px + 24 * pix, flops=forward + 400 * vertices)
    if kind == "batch":
        return dict(bytes=mesh + 2 * maps + n * (12 * px + 24 * pix), flops=n * (forward + 600 * vertices))
    if kind == "objective":
        taps = (2 * case["radius"] + 1) ** 2
        return dict(bytes=mesh + 2 * maps + pix * (32 + 12 * 4), flops=pix * (ray + 3 * taps * 41))
    return dict(bytes=2 * mesh + 12 * tex + 32 * pix, flops=pix * ray + 50 * tris * math.log2(max(tris, 2)))


# ------------------------------------------------------------------ the same in 64 bits
# A plain path tracer in torch, every ray against every triangle, gradients by torch's own
# autograd with the sampled directions and their densities held constant.

F64 = torch.float64
PI = math.pi
M32 = 0xffffffff


def _t(x):
    return torch.as_tensor(np.asarray(x, np.float64), dtype=F64, device="cuda")


def _philox(pixel, sample, block, key):
    """Philox4x32-10 on int64 tensors holding 32-bit words."""
    c = [pixel, sample, torch.full_like(pixel, block), torch.zeros_like(pixel)]
    k0, k1 = key & M32, (key >> 32) & M32
    for _ in range(10):
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57   # low 64 bits of each product
        c = [((p1 >> 32) & M32) ^ c[1] ^ k0, p1 & M32, ((p0 >> 32) & M32) ^ c[3] ^ k1, p0 & M32]
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return [(x >> 8).to(F64) / 16777216.0 for x in c]


def _dot(a, b):
    return (a * b).sum(-1)


def _unit(a):
    return a / _dot(a, a).sqrt()[..., None]


def _hits(P, o, d, tmin, skip, tmax=None):
    """Closest triangle (index, -1: none) per ray, or whether any lies before tmax."""
    n, T = o.shape[0], P.shape[0]
    best = torch.full((n,), -1, dtype=torch.long, device=o.device)
    near = torch.full((n,), math.inf, dtype=F64, device=o.device) if tmax is None else tmax.clone()
    step = max(1, int(1 << 25) // max(n, 1))
    for t0 in range(0, T, step):
        v0, v1, v2 = P[t0:t0 + step].unbind(1)
        e1, e2 = v1 - v0, v2 - v0
        # Cramer's rule, its triple products expanded so each is one small matrix product
        nrm = torch.linalg.cross(e1, e2)
        det = -(d @ nrm.T)
        m = torch.linalg.cross(o, d)   # o x d: the ray's moment
        w0 = torch.linalg.cross(v0, e2)
        w1 = torch.linalg.cross(v0, e1)
        b1 = (m @ e2.T + d @ w0.T) / det
        b2 = -(m @ e1.T + d @ w1.T) / det
        t = (o @ nrm.T - _dot(v0, nrm)) / det
        ok = (b1 >= 0) & (b2 >= 0) & (b1 + b2 <= 1) & (t > tmin)
        ok &= torch.arange(t0, t0 + v0.shape[0], device=o.device)[None] != skip[:, None]
        tt, k = torch.where(ok, t, math.inf).min(1)
        take = tt < near
        near = torch.where(take, tt, near)
        best = torch.where(take, k + t0, best)
    return best


def _rays(P, o, d, tmin, skip, tmax=None):
    """_hits in pieces of rays."""
    out = []
    for k in range(0, o.shape[0], 1 << 20):
        s = slice(k, k + (1 << 20))
        out.append(_hits(P, o[s], d[s], tmin, skip[s], None if tmax is None else tmax[s]))
    return torch.cat(out)


def _lookup(m, x, y):
    """Bilinear, clamp to edge; x, y in texels with texel centres at integers."""
    H, W = m.shape[:2]
    fx, fy = x.floor(), y.floor()
    ax, ay = x - fx, y - fy
    if m.dim() == 3:
        ax, ay = ax[:, None], ay[:, None]
    cl = lambda v, n: v.long().clamp(0, n - 1)
    x0, x1, y0, y1 = cl(fx, W), cl(fx + 1, W), cl(fy, H), cl(fy + 1, H)
    return (m[y0, x0] * (1 - ax) * (1 - ay) + m[y0, x1] * ax * (1 - ay) + m[y1, x0] * (1 - ax) * ay
            + m[y1, x1] * ax * ay)


def _to_world(n, x, y, z):
    s = torch.copysign(torch.ones_like(n[:, 2]), n[:, 2])
    a = -1 / (s + n[:, 2])
    b = n[:, 0] * n[:, 1] * a
    t1 = torch.stack([1 + s * n[:, 0] ** 2 * a, s * b, -s * n[:, 0]], -1)
    t2 = torch.stack([b, s + n[:, 1] ** 2 * a, -n[:, 1]], -1)
    return t1 * x[:, None] + t2 * y[:, None] + n * z[:, None]


def _cosine(n, u1, u2):
    r = u1.sqrt()
    return _to_world(n, r * torch.cos(2 * PI * u2), r * torch.sin(2 * PI * u2), (1 - u1).sqrt())


def _alpha(r):
    return (r * r).clamp_min(1e-3)


def _reflect(kind, n, wo, wi, alb, r, sp):
    """albedo / pi + F D G / (4 cos cos), 0 below the surface."""
    ci, co = _dot(n, wi), _dot(n, wo)
    on = (ci > 0) & (co > 0)
    f = alb / PI
    if kind == GGX:
        h = _unit(wi + wo)
        a2 = _alpha(r) ** 2
        nh2 = _dot(n, h) ** 2
        c = torch.linalg.cross(n, h)
        D = a2 / (PI * (a2 * nh2 + _dot(c, c)) ** 2)
        ci1, co1 = torch.where(on, ci, 1.0), torch.where(on, co, 1.0)
        g = lambda x: 2 * x / (x + (a2 + (1 - a2) * x * x).sqrt())
        F0 = 0.08 * sp
        F = F0 + (1 - F0) * (1 - _dot(wi, h)) ** 5
        f = f + (F * D * g(ci1) * g(co1) / (4 * ci1 * co1))[:, None]
    return torch.where(on[:, None], f, 0.0)


def _bounce(kind, n, wo, r, u):
    wi = _cosine(n, u[1], u[2])
    pd = lambda w: _dot(n, w).clamp_min(0) / PI
    if kind == LAMBERT:
        return wi, pd(wi)
    a = _alpha(r)
    t2 = a * a * u[1] / (1 - u[1])
    ct = 1 / (1 + t2).sqrt()
    st = t2.sqrt() * ct
    h = _to_world(n, st * torch.cos(2 * PI * u[2]), st * torch.sin(2 * PI * u[2]), ct)
    ws = h * (2 * _dot(wo, h))[:, None] - wo
    wi = torch.where((u[0] < 0.25)[:, None], ws, wi)
    v = wi + wo
    h = _unit(v)
    nh, oh = _dot(n, h).abs(), _dot(wo, h).abs()
    c = torch.linalg.cross(n, h)
    D = a * a / (PI * (a * a * nh * nh + _dot(c, c)) ** 2)
    ps = torch.where((nh > 0) & (oh > 0), D * nh / (4 * oh), 0.0)
    return wi, 0.75 * pd(wi) + 0.25 * ps


class _Exact:
    """The workload's geometry and cameras in 64 bits."""

    def __init__(self, case, w, verts=None):
        self.case, self.w = case, w
        V = _t(w.mesh.vertices if verts is None else verts)
        F = torch.as_tensor(w.mesh.triangles.astype(np.int64)).cuda()
        self.P = V[F]
        self.uv = _t(w.mesh.corner_uvs)
        lo, hi = w.mesh.vertices.astype(np.float64).min(0), w.mesh.vertices.astype(np.float64).max(0)
        self.tmin = float(np.float32(1e-5 * math.sqrt(((hi - lo) ** 2).sum())))
        c, p = w.camera, w.projector
        self.M = _t(c.R.T @ np.linalg.inv(c.K))
        self.o = _t(-c.R.T @ c.t)
        self.pR, self.pt, self.pK, self.po = _t(p.R), _t(p.t), _t(p.K), _t(-p.R.T @ p.t)

    def camera(self, x, y):
        d = _unit(torch.stack([x, y, torch.ones_like(x)], -1) @ self.M.T)
        return self.o.expand_as(d), d

    def surface(self, k, o, d):
        v0, v1, v2 = self.P[k].unbind(1)
        e1, e2 = v1 - v0, v2 - v0
        p = torch.linalg.cross(d, e2)
        det = _dot(e1, p)
        tv = o - v0
        b1, b2 = _dot(tv, p) / det, _dot(d, torch.linalg.cross(tv, e1)) / det
        b = torch.stack([1 - b1 - b2, b1, b2], -1)
        x = (self.P[k] * b[..., None]).sum(1)
        n = _unit(torch.linalg.cross(e1, e2))
        n = torch.where((_dot(n, d) > 0)[:, None], -n, n)
        return x, n, (self.uv[k] * b[..., None]).sum(1)

    def render(self, proj, alb, rough, spec, scal):
        """The image; differentiable in the five tensors."""
        w, case = self.w, self.case
        H, W, spp = case["ch"], case["cw"], case["spp"]
        gp, mix, gc, wb = scal[0:3], scal[3:12].reshape(3, 3), scal[12:15], scal[15:18]
        y = torch.where(proj > 0, proj.clamp_min(1e-300) ** gp, 0.0)
        Ep = (w.prf_gain * (y @ mix.T)).clamp_min(0)
        env = _t(w.env)
        thr = w.clip_k / wb.min()
        rows = max(1, (1 << 17) // (W * spp))   # image rows in flight
        img = []
        for y0 in range(0, H, rows):
            y1 = min(H, y0 + rows)
            g = torch.arange(y0 * W * spp, y1 * W * spp, device="cuda")
            if torch.is_grad_enabled():
                L = torch.utils.checkpoint.checkpoint(self._radiance, g, Ep, alb, rough, spec, env, use_reentrant=False)
            else:
                L = self._radiance(g, Ep, alb, rough, spec, env)
            if w.clip:
                L = torch.minimum(L, thr)
            E = L.reshape(y1 - y0, W, spp, 3).mean(2)
            v = w.crf_gain * wb * E
            img.append(torch.where(v > 0, torch.where(v > 0, v, 1.0) ** gc, 0.0))
        return torch.cat(img)

    def _radiance(self, g, Ep, alb, rough, spec, env):
        w, kind = self.w, self.case["brdf"]
        spp, W = self.case["spp"], self.case["cw"]
        key = int(w.seed)
        pixel, smp = g // spp, g % spp + w.sample_offset
        u = _philox(pixel, smp, 0, key)
        o, d = self.camera((pixel % W).to(F64) + u[0], (pixel // W).to(F64) + u[1])
        L = torch.zeros((g.numel(), 3), dtype=F64, device="cuda")
        beta = torch.ones_like(L)
        idx = torch.arange(g.numel(), device="cuda")
        skip = torch.full_like(idx, -1)
        for depth in range(self.case["depth"]):
            k = _rays(self.P, o, d, self.tmin, skip)
            if depth == 0:
                L = L + torch.where((k < 0)[:, None], env, 0.0)
            on = k >= 0
            idx, k, o, d, beta = idx[on], k[on], o[on], d[on], beta[on]
            if idx.numel() == 0:
                break
            x, n, uv = self.surface(k, o, d)
            wo = -d
            tx, ty = uv[:, 0] * alb.shape[1] - 0.5, uv[:, 1] * alb.shape[0] - 0.5
            a = _lookup(alb, tx, ty)
            r = _lookup(rough, tx, ty)
            sp = _lookup(spec, tx, ty)
            # the projector
            xp = x @ self.pR.T + self.pt
            q = xp @ self.pK.T
            pu, pv = q[:, 0] / xp[:, 2], q[:, 1] / xp[:, 2]
            tow = self.po - x
            dist = _dot(tow, tow).sqrt()
            wp = tow / dist[:, None]
            cp = _dot(n, wp)
            lit = (xp[:, 2] > 0) & (pu >= 0) & (pu < Ep.shape[1]) & (pv >= 0) & (pv < Ep.shape[0]) & (cp > 0)
            j = lit.nonzero()[:, 0]
            j = j[_rays(self.P, x[j], wp[j], self.tmin, k[j], dist[j] - self.tmin) < 0]
            ca = xp[j, 2] / _dot(xp[j], xp[j]).sqrt()
            geom = cp[j] / (ca ** 3 * dist[j] ** 2)
            f = _reflect(kind, n[j], wo[j], wp[j], a[j], r[j], sp[j])
            E = _lookup(Ep, pu[j] - 0.5, pv[j] - 0.5)
            L = L.index_add(0, idx[j], beta[j] * f * E * geom[:, None])
            # the environment
            if bool((env != 0).any()):
                u = _philox(pixel[idx], smp[idx], 2 + 2 * depth, key)
                we = _cosine(n, u[0], u[1])
                j = (_rays(self.P, x, we, self.tmin, k, torch.full_like(dist, math.inf)) < 0).nonzero()[:, 0]
                f = _reflect(kind, n[j], wo[j], we[j], a[j], r[j], sp[j])
                L = L.index_add(0, idx[j], beta[j] * f * env * PI)
            if depth == self.case["depth"] - 1:
                break
            u = _philox(pixel[idx], smp[idx], 1 + 2 * depth, key)
            with torch.no_grad():
                wi, pdf = _bounce(kind, n, wo, r, u)
                ci = _dot(n, wi)
                j = ((ci > 0) & (pdf > 0)).nonzero()[:, 0]
            f = _reflect(kind, n[j], wo[j], wi[j], a[j], r[j], sp[j])
            beta = beta[j] * f * (ci[j] / pdf[j])[:, None]
            idx, o, d, skip = idx[j], x[j], wi[j], k[j]
        return L

    def gbuffer(self, alb):
        H, W = self.case["ch"], self.case["cw"]
        g = torch.arange(H * W, device="cuda")
        o, d = self.camera((g % W).to(F64) + 0.5, (g // W).to(F64) + 0.5)
        k = _rays(self.P, o, d, self.tmin, torch.full_like(g, -1))
        on = k >= 0
        x, n, uv = self.surface(k.clamp_min(0), o, d)
        a = _lookup(alb, uv[:, 0] * alb.shape[1] - 0.5, uv[:, 1] * alb.shape[0] - 0.5)
        out = torch.cat([a, n, _dot(x - o, d)[:, None], torch.ones_like(a[:, :1])], -1)
        return torch.where(on[:, None], out, 0.0).reshape(H, W, 8)


def _denoise(img, guide, cfg):
    H, W = img.shape[:2]
    a = _t(np.asarray(cfg.guide, np.float32))
    spatial = float(np.float32(cfg.spatial))
    num, den = torch.zeros_like(img), torch.zeros_like(img[..., :1])
    for dy in range(-cfg.radius, cfg.radius + 1):
        for dx in range(-cfg.radius, cfg.radius + 1):
            if abs(dy) >= H or abs(dx) >= W:
                continue
            ys, xs = slice(max(0, -dy), H - max(0, dy)), slice(max(0, -dx), W - max(0, dx))
            yq, xq = slice(max(0, dy), H + min(0, dy)), slice(max(0, dx), W + min(0, dx))
            e = spatial * (dx * dx + dy * dy) + (a * (guide[ys, xs] - guide[yq, xq]) ** 2).sum(-1)
            wt = torch.exp(-e)[..., None]
            pad = (0, 0, max(0, -dx), max(0, dx), max(0, -dy), max(0, dy))
            num = num + torch.nn.functional.pad(wt * img[yq, xq], pad)
            den = den + torch.nn.functional.pad(wt, pad)
    return num / den


def _tv(m):
    return (m[1:] - m[:-1]).abs().mean() + (m[:, 1:] - m[:, :-1]).abs().mean()


def exact(case, seed):
    kind = case["kind"]
    tris = 14 if case["quads"] == 0 else 4 * case["quads"] ** 2 + 36
    paths = case["cw"] * case["ch"] * case["pairs"] * (case["spp"] if kind not in ("build", "objective") else 1)
    # brute force: a few 1e11 ray-triangle tests at most; the metallic / normal-map shading,
    # the pose gradient and the refitted surface have no 64-bit form here
    if kind in ("pose", "refit") or case["ext"] or paths * tris > 2e10 or (kind not in ("build", "objective") and
                                                                        paths * case["depth"] * tris > 4e9):
        return None
    w, rng = _workload(case, seed)
    x = _Exact(case, w)
    H, W = case["ch"], case["cw"]
    maps = [_t(w.albedo), _t(w.roughness), _t(w.specular)]
    proj = _t(w.proj_image)
    scal = _t(np.concatenate([np.ravel(w.prf_gamma), np.ravel(w.prf_mix), np.ravel(w.crf_gamma),
                              np.ravel(w.white_balance)]).astype(np.float32))
    f32 = lambda a: _t(np.ascontiguousarray(a, np.float32))
    if kind == "build":
        with torch.no_grad():
            return x.gbuffer(maps[0])
    if kind == "relight":
        with torch.no_grad():
            return x.render(proj, *maps, scal)
    if kind == "step":
        G = f32(rng.normal(size=(H, W, 3)))
        leaves = [t.requires_grad_(True) for t in [proj] + maps + [scal]]
        img = x.render(*leaves)
        g = torch.autograd.grad((img * G).sum(), leaves, allow_unused=True)
        g = [torch.zeros_like(t) if v is None else v for t, v in zip(leaves, g)]
        names = ["d_proj_image", "d_albedo", "d_roughness", "d_specular", "d_scalars"]
        out = dict(zip(names, g))
        return out if case["mode"] == "own" else dict(image=img.detach(), **out)
    if kind in ("fit", "compensate"):
        target = f32(rng.uniform(0, 1, (H, W, 3)))
        leaves = maps + [scal] if kind == "fit" else [proj]
        for t in leaves:
            t.requires_grad_(True)
        img = x.render(proj, *maps, scal)
        g = torch.autograd.grad(((img - target) ** 2).mean(), leaves)
        return dict(image=img.detach(), grads=list(g))
    if kind == "batch":
        images = [f32(rng.uniform(0, 1, (case["ph"], case["pw"], 3))) for _ in range(case["pairs"])]
        targets = [f32(rng.uniform(0, 1, (H, W, 3))) for _ in range(case["pairs"])]
        leaves = [t.requires_grad_(True) for t in maps + [scal]]
        outs, total = [], [torch.zeros_like(t) for t in leaves]
        for ip, tgt in zip(images, targets):
            img = x.render(ip, *leaves)
            g = torch.autograd.grad(((img - tgt) ** 2).mean(), leaves)
            outs.append(img.detach())
            total = [a + b / case["pairs"] for a, b in zip(total, g)]
        return dict(images=outs, grads=dict(zip(["d_albedo", "d_roughness", "d_specular", "d_scalars"], total)))
    # objective
    image, target = f32(rng.uniform(0, 1, (H, W, 3))), f32(rng.uniform(0, 1, (H, W, 3)))
    with torch.no_grad():
        guide = x.gbuffer(maps[0])
    leaves = [t.requires_grad_(True) for t in [image] + maps]
    loss = (_denoise(image, guide, objective.DenoiseConfig(radius=case["radius"])) - target).abs().mean()
    loss = loss + 0.1 * sum(_tv(m) for m in maps)
    return dict(loss=loss.detach(), guide=guide, grads=list(torch.autograd.grad(loss, leaves)))
