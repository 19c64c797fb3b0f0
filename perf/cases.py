"""The work that programs built on this framework have it do, as cases that can be timed.

Each listed case is one call (or one short sequence of calls) of the public Python entry
points, at sizes of the repository's own workloads and tests:

* one captured fit step (``FitStep.replay``) from a freshly reloaded Gaussian set, from the
  smallest set (1,000 Gaussians, one 128 x 128 view) to the foveal refinement of 500,000
  Gaussians over 16 views of 1920 x 1920;
* the differentiable rasterizer inside a PyTorch program (``rasterize`` and its backward);
* forward rendering alone (``Plan.forward``), as a viewer calls it;
* the steps around the fit: ray-marched targets, Gaussians seeded from the volume, the
  first-hit point cloud, and the viewer's reprojection warp.

``listed()`` names them, ``draw(rng)`` gives further ones of the same ranges, ``prepare``
makes what a program holds before the call, ``run`` is the call, ``work`` the bytes and
operations it cannot do without, and ``exact`` its result in 64 bits.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2601_22026_amd as gs

DEV = "cuda:0"
Y00 = 0.5 / math.sqrt(math.pi)                 # the constant spherical-harmonic basis function
THRESHOLD, RANGE, EXTINCTION = 1200.0, 1800.0, 40.0   # transfer function of the volume
TF_LO, TF_HI = (0.8, 0.3, 0.2), (1.0, 0.95, 0.9)
T_STOP = 1e-4
RADIUS = 0.2                                   # fovea radius as a fraction of the view's width
HIT_ALPHA, COLOR_STEPS, HIT_STEP = 0.5, 8, 0.01


# ---- the cases ------------------------------------------------------------------------

def listed():
    uneven = "512x512,768x1024,1024x1024,1536x1536,768x1024,2048x2048,512x512,1024x1024"
    return [
        # the smallest fit: latency and launches are all there is
        dict(name="fit_small", do="fit", n=1000, sh=0, scene="random", sizes="128x128",
             tile=16, batch=128, t_mode=1),
        # the initial fit of the paper's shape: 20,000 Gaussians, one 512 x 512 view a step
        dict(name="fit_initial", do="fit", n=20000, sh=0, scene="phantom", volume=128,
             sizes="512x512", tile=16, batch=128, t_mode=1),
        # the phantom fit: 50,000 Gaussians crowded in the middle of one 1024 x 1024 view
        dict(name="fit_phantom", do="fit", n=50000, sh=0, scene="phantom", volume=128,
             sizes="1024x1024", tile=16, batch=64, t_mode=1),
        # alpha training over random backgrounds with the visibility-masked optimiser, views
        # of odd sizes, colour of first degree
        dict(name="fit_alpha", do="fit", n=60001, sh=1, scene="phantom", volume=96,
             sizes="799x601,640x480,333x517", tile=16, batch=128, t_mode=1, alpha=True),
        # many uneven views at once, colour of third degree
        dict(name="fit_batched", do="fit", n=200000, sh=3, scene="random", sizes=uneven,
             tile=16, batch=128, t_mode=0),
        # the foveal refinement, the headline workload: only the fovea disks carry loss
        dict(name="fit_foveal", do="fit", n=500000, sh=0, scene="phantom", volume=256,
             sizes=",".join(["1920x1920"] * 16), tile=16, batch=64, t_mode=0, gaze=True),
        # the rasterizer as one operation of a PyTorch program, an odd view
        dict(name="autograd_odd", do="autograd", n=30011, sh=2, scene="random", sizes="701x533",
             tile=16, batch=128, t_mode=0),
        # a viewer's stereo frame of a large model, forward alone
        dict(name="render_stereo", do="render", n=1000000, sh=3, scene="random",
             sizes="2064x2208,2064x2208", tile=16, batch=128, t_mode=0),
        # the target images of a fit, marched through the volume
        dict(name="raymarch", do="raymarch", volume=256,
             sizes="1024x1024,1024x1024,1024x1024,1024x1024"),
        # a regeneration's first step: Gaussians from the resident volume
        dict(name="seed_volume", do="seed", volume=256, cap=500000),
        # the initial point cloud: first hits of the rays of 8 views
        dict(name="first_hits", do="hits", volume=128, sizes=",".join(["256x256"] * 8), cap=20000),
        # the viewer's foveal image moved to the next head pose
        dict(name="warp_eye", do="warp", sizes="2064x2208", out="2064x2208"),
    ]


def _span(rng, lo, hi):
    """An integer of [lo, hi], spread over its logarithm; odd as often as even."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _text(sizes):
    return ",".join("%dx%d" % s for s in sizes)


def draw(rng):
    do = rng.choice(["fit", "fit", "fit", "fit", "foveal", "autograd", "render", "raymarch", "seed",
                     "hits", "warp"])
    tile = rng.choice([16, 16, 16, 16, 8])
    plan = dict(tile=tile, batch=rng.choice([64, 128]), t_mode=rng.choice([0, 1]))
    if do in ("fit", "autograd"):
        n = _span(rng, 800, 200000)
        views = rng.choice([1, 1, 1, 2, 3, 4, 6]) if do == "fit" else rng.choice([1, 2])
        sizes = [(_span(rng, 96, 1400), _span(rng, 96, 1400)) for _ in range(views)]
        scene = rng.choice(["random", "phantom"])
        case = dict(do=do, n=n, sh=rng.choice([0, 0, 1, 2, 3]), scene=scene, sizes=_text(sizes), **plan)
        if scene == "phantom":
            case["volume"] = rng.choice([64, 96, 128])
        if do == "fit" and rng.random() < 0.25:
            case["alpha"] = True
        return case
    if do == "foveal":
        side = _span(rng, 512, 1920)
        return dict(do="fit", n=_span(rng, 40000, 400000), sh=0, scene="phantom", volume=192,
                    sizes=_text([(side, side)] * rng.choice([2, 4, 8, 12])), gaze=True, **plan)
    if do == "render":
        return dict(do=do, n=_span(rng, 5000, 800000), sh=rng.choice([0, 1, 3]), scene="random",
                    sizes=_text([(_span(rng, 400, 2000), _span(rng, 400, 2000))] * rng.choice([1, 2])),
                    **plan)
    if do == "raymarch":
        return dict(do=do, volume=rng.choice([64, 97, 128, 200, 256]),
                    sizes=_text([(_span(rng, 128, 1100), _span(rng, 128, 1100))
                                 for _ in range(rng.choice([1, 2, 4]))]))
    if do == "seed":
        return dict(do=do, volume=_span(rng, 64, 256), cap=_span(rng, 5000, 500000))
    if do == "hits":
        side = _span(rng, 100, 400)
        return dict(do=do, volume=rng.choice([64, 100, 128]), sizes=_text([(side, side)] * rng.choice([4, 8])),
                    cap=_span(rng, 2000, 40000))
    w, h = _span(rng, 300, 2064), _span(rng, 300, 2208)
    return dict(do=do, sizes="%dx%d" % (w, h), out="%dx%d" % (_span(rng, 300, w + 64), h))


def _sizes(case):
    return [tuple(int(x) for x in s.split("x")) for s in case["sizes"].split(",")]


# ---- inputs, made on the GPU from the seed alone ---------------------------------------

def _gen(seed, stream):
    return torch.Generator(device=DEV).manual_seed((int(seed) * 1000003 + stream * 7919) & 0x7FFFFFFF)


def _volume(n, seed):
    """A CT-like uint16 volume (stored as int16): 20 ellipsoids of HU-like values plus noise."""
    g = _gen(seed, 1)
    c = (torch.arange(n, device=DEV) + 0.5) * (2.0 / n) - 1.0
    ctr = torch.rand(20, 3, device=DEV, generator=g) * 1.2 - 0.6
    axes = torch.rand(20, 3, device=DEV, generator=g) * 0.4 + 0.1
    rot = torch.linalg.qr(torch.randn(20, 3, 3, device=DEV, generator=g).cpu())[0].to(DEV)
    val = torch.rand(20, device=DEV, generator=g) * 1200.0 + 400.0
    vol = torch.randn(n, n, n, device=DEV, generator=g) * 20.0
    for e in range(20):
        M = rot[e] / axes[e]                       # [3][3]: world axis -> scaled ellipsoid axis
        d = [(c - ctr[e, a])[:, None] * M[a] for a in range(3)]
        q = torch.zeros(n, n, n, device=DEV)
        for k in range(3):
            q += (d[0][:, None, None, k] + d[1][None, :, None, k] + d[2][None, None, :, k]) ** 2
        vol += val[e] * (q <= 1.0)
    return vol.clamp_(0.0, 3000.0).round_().to(torch.int16)


def _camera(center, target, width, height, fov=60.0):
    c = np.asarray(center, np.float64)
    f = np.asarray(target, np.float64) - c
    f /= np.linalg.norm(f)
    up = np.array([0.0, -1.0, 0.0]) if abs(f[1]) < 0.99 else np.array([0.0, 0.0, 1.0])
    x = np.cross(f, up)
    x /= np.linalg.norm(x)
    R = np.stack([x, np.cross(f, x), f]).astype(np.float32)
    fx = float(np.float32(0.5 * width / math.tan(math.radians(fov) / 2)))
    return SimpleNamespace(R=R, t=(-(R.astype(np.float64) @ c)).astype(np.float32),
                           campos=c.astype(np.float32), fx=fx, fy=fx, cx=width / 2.0, cy=height / 2.0,
                           tanx=float(np.float32(0.5 * width / fx)), tany=float(np.float32(0.5 * height / fx)),
                           znear=float(np.float32(0.2)), bg=np.zeros(3, np.float32), width=width, height=height)


def _cameras(case, seed):
    """Views on the radius-3 sphere, looking at the middle; a stereo pair where a viewer renders."""
    rng = np.random.default_rng([int(seed), 2])
    sizes, cams = _sizes(case), []
    for k, (w, h) in enumerate(sizes):
        if k and case["do"] == "render":
            c = cams[0].campos.astype(np.float64) + 0.064 * cams[0].R[0]
            cams.append(_camera(c, c + cams[0].R[2], w, h))
            continue
        d = rng.normal(size=3)
        cams.append(_camera(3.0 * d / np.linalg.norm(d), (0.0, 0.0, 0.0), w, h))
    return cams


def _gaussians(case, seed):
    """Planar float32 [C][n]: random ones (constant overlap as n grows), or voxels of the phantom
    above the threshold, one voxel wide, as a fit a few hundred steps on has them."""
    n, K = case["n"], (case["sh"] + 1) ** 2
    g = _gen(seed, 3)

    def rand(*s):
        return torch.rand(*s, device=DEV, generator=g)

    def randn(*s):
        return torch.randn(*s, device=DEV, generator=g)

    P = torch.zeros(11 + 3 * K, n, device=DEV)
    if case["scene"] == "random":
        P[0:3] = rand(3, n) * 2.0 - 1.0
        P[3:6] = -3.0 - math.log(n / 1000.0) / 3.0 + 0.5 * randn(3, n)
        P[10] = randn(n)
        P[11:14] = (rand(3, n) - 0.5) / Y00
    else:
        m = case["volume"]
        vol = _volume(m, seed).reshape(-1)
        at = torch.nonzero(vol > THRESHOLD).reshape(-1)
        at = at[torch.randint(at.numel(), (n,), device=DEV, generator=g).sort().values]
        t = ((vol[at].float() - THRESHOLD) / RANGE).clamp(0.0, 1.0)
        for a, i in enumerate((at // (m * m), at // m % m, at % m)):
            P[a] = (i + 0.5) * (2.0 / m) - 1.0 + (rand(n) - 0.5) * (1.0 / m)
        P[3:6] = math.log(2.0 / m) + 0.2 * randn(3, n)
        P[10] = math.log(0.1 / 0.9) + 0.5 * randn(n)
        for c in range(3):
            P[11 + c] = (TF_LO[c] * (1 - t) + TF_HI[c] * t - 0.5) / Y00
    P[6:10] = randn(4, n)
    P[6:10] /= P[6:10].norm(dim=0, keepdim=True)
    if K > 1:
        P[14:] = 0.05 * randn(3 * (K - 1), n)
    return P


def _targets(case, seed):
    """Per view a smooth random image with a little noise (premultiplied RGBA for alpha training),
    views concatenated."""
    g, planes, out = _gen(seed, 4), 4 if case.get("alpha") else 3, []
    for w, h in _sizes(case):
        low = torch.rand(1, planes, 12, 12, device=DEV, generator=g)
        img = torch.nn.functional.interpolate(low, size=(h, w), mode="bilinear")[0]
        img = (img * 0.9 + 0.1 * torch.rand(planes, h, w, device=DEV, generator=g)).contiguous()
        if planes == 4:
            img[:3] *= img[3]
        out.append(img.reshape(-1))
    return torch.cat(out)


def _gaze(case, seed):
    rng = np.random.default_rng([int(seed), 5])
    return np.array([(rng.uniform(0.2, 0.8) * w, rng.uniform(0.2, 0.8) * h) for w, h in _sizes(case)],
                    np.float32)


def _clip_matrices(cam, near=0.1, far=100.0):
    P, V = np.zeros((4, 4)), np.eye(4)
    P[0, 0], P[0, 2] = 2 * cam.fx / cam.width, 2 * cam.cx / cam.width - 1
    P[1, 1], P[1, 2] = 2 * cam.fy / cam.height, 2 * cam.cy / cam.height - 1
    P[2, 2], P[2, 3], P[3, 2] = (far + near) / (far - near), -2 * far * near / (far - near), 1.0
    V[:3, :3], V[:3, 3] = cam.R, cam.t
    return P.astype(np.float32), V.astype(np.float32)


def _warp_inputs(case, seed):
    """An eye's image with the first-hit distance of a unit sphere (no depth where a ray misses),
    and the head pose a frame later."""
    (w, h), rng = _sizes(case)[0], np.random.default_rng([int(seed), 6])
    old = _camera((0.2, -0.1, -2.5), rng.uniform(-0.05, 0.05, 3), w, h)
    new = _camera(np.array((0.2, -0.1, -2.5)) + rng.uniform(-0.03, 0.03, 3), rng.uniform(-0.05, 0.05, 3), w, h)
    f64 = dict(dtype=torch.float64, device=DEV)
    x = (torch.arange(w, **f64) + 0.5 - old.cx) / old.fx
    y = (torch.arange(h, **f64) + 0.5 - old.cy) / old.fy
    d = torch.stack([x[None, :].expand(h, w), y[:, None].expand(h, w), torch.ones(h, w, **f64)], -1)
    d = d @ torch.from_numpy(old.R.astype(np.float64)).to(DEV)
    d /= d.norm(dim=-1, keepdim=True)
    o = torch.from_numpy(old.campos.astype(np.float64)).to(DEV)
    b = d @ o
    disc = b * b - (o @ o - 1.0)
    t = -b - disc.clamp(min=0).sqrt()
    depth = torch.where((disc > 0) & (t > 0), t, torch.zeros_like(t)).float()
    rgba = torch.rand(4, h, w, device=DEV, generator=_gen(seed, 7))
    return old, new, depth.contiguous(), rgba


_STREAM = []


def _stream():
    """The program's one stream (a graph cannot be captured on the null stream)."""
    if not _STREAM:
        _STREAM.append(torch.cuda.Stream())
    return _STREAM[0]


def prepare(case, seed):
    do = case["do"]
    s = dict(do=do, stream=_stream())
    with torch.cuda.stream(s["stream"]):
        ctx = s["ctx"] = gs.Context(0)
        if do in ("fit", "autograd", "render"):
            P, cams = _gaussians(case, seed), _cameras(case, seed)
            s["P"] = P
            if do == "fit":
                gaze = torch.from_numpy(_gaze(case, seed)).to(DEV) if case.get("gaze") else None
                alpha = bool(case.get("alpha"))
                cfg = gs.FitConfig(tile=case["tile"], lds_batch=case["batch"], t_mode=case["t_mode"],
                                   radius_frac=RADIUS, fovea_cull=gaze is not None, alpha_loss=alpha,
                                   random_bg=alpha, masked_adam=alpha, bg_seed=int(seed))
                s["fit"] = gs.FitStep(ctx, P.clone(), cams, _targets(case, seed), gaze, cfg=cfg)
                s["fit"].capture()
            else:
                s["cams"] = gs.cameras_to_device(cams, DEV)
                keys = gs.measure_keys(ctx, P, s["cams"], _sizes(case), case["sh"], case["tile"])
                s["plan"] = gs.Plan(ctx, case["n"], _sizes(case), case["sh"], case["tile"], case["batch"],
                                    t_mode=case["t_mode"], key_capacity=keys * 5 // 4 + 65536)
                if do == "autograd":
                    s["g"] = torch.randn(4 * s["plan"].total_pixels, device=DEV, generator=_gen(seed, 8))
                else:
                    s["rgba"] = torch.zeros(4 * s["plan"].total_pixels, device=DEV)
        elif do in ("raymarch", "seed", "hits"):
            s["vol"] = _volume(case["volume"], seed)
            s["seed"] = int(seed)
            if do != "seed":
                s["cams"] = _cameras(case, seed)
            if do == "raymarch":
                s["rgba"] = torch.zeros(4 * sum(w * h for w, h in _sizes(case)), device=DEV)
            else:
                s["cap"] = case["cap"]
        else:
            old, new, s["depth"], s["rgba"] = _warp_inputs(case, seed)
            s["poses"] = (*_clip_matrices(old), old.campos, *_clip_matrices(new))
            s["out"] = tuple(int(x) for x in case["out"].split("x"))
            s["zbuf"] = torch.empty(s["out"][0] * s["out"][1], dtype=torch.int64, device=DEV)
        s["stream"].synchronize()
    return s


def run(s):
    with torch.cuda.stream(s["stream"]):
        do = s["do"]
        if do == "fit":
            # the refinement's restart (the Gaussians reloaded, the optimiser's state discarded)
            # and one step from there, so that every pass does the same work
            fit = s["fit"]
            fit.restart(s["P"])
            fit.replay()
            return dict(loss=fit.loss, rgba=fit.rgba, grads=fit.grads, m=fit.m, v=fit.v)
        if do == "autograd":
            P = s["P"].detach().requires_grad_()
            img = gs.rasterize(P, s["plan"], s["cams"])
            (grads,) = torch.autograd.grad(img, P, s["g"])
            return dict(rgba=img.detach(), grads=grads)
        if do == "render":
            s["plan"].forward(s["P"], s["P"].shape[1], s["cams"], s["rgba"])
            return s["rgba"]
        if do == "raymarch":
            return gs.raymarch(s["ctx"], s["vol"], s["cams"], out=s["rgba"])
        if do == "seed":
            return gs.seed_volume(s["ctx"], s["vol"], cap=s["cap"], seed=s["seed"])
        if do == "hits":
            P, rays = gs.seed_first_hits(s["ctx"], s["vol"], s["cams"], s["cap"], s["seed"], HIT_STEP,
                                         hit_alpha=HIT_ALPHA, color_steps=COLOR_STEPS)
            return dict(params=P, rays=rays)
        rgba, src = gs.reproject_warp(s["ctx"], s["rgba"], s["depth"], *s["poses"], *s["out"],
                                      zbuf=s["zbuf"])
        return dict(rgba=rgba, src=src)


_SAMPLES = 0.9   # ray-march samples per voxel edge and ray


def _pairs(case):
    """Pairs of a splat and a pixel that the image includes, which compositing cannot do without:
    footprints times Gaussians, up to the depth at which pixels stop (both as Plan.count_pairs has
    them on the listed scenes)."""
    n, total = case["n"], 0.0
    for w, h in _sizes(case):
        if case["scene"] == "random":
            total += min(175.0 * (w * h / 128.0 ** 2) * (n / 1000.0) ** (-2 / 3) * n, 38.0 * w * h)
        else:
            most = 115.0 * (w * h / 512.0 ** 2) * (128.0 / case["volume"]) ** 2 * n
            disk = math.pi * (RADIUS * w) ** 2
            total += min(0.26 * most, 120.0 * disk) if case.get("gaze") else min(most, 60.0 * w * h)
    return total


def work(case):
    do = case["do"]
    sizes = _sizes(case) if "sizes" in case else []
    pix = sum(w * h for w, h in sizes)
    if do in ("fit", "autograd", "render"):
        elems = (11 + 3 * (case["sh"] + 1) ** 2) * case["n"]
        if case.get("gaze"):
            pix = sum(math.pi * (RADIUS * w) ** 2 for w, _ in sizes)
        pairs = _pairs(case)
        if do == "render":
            return dict(bytes=4 * elems + 16 * pix, flops=28 * pairs)
        if do == "autograd":     # parameters in, image out, its gradient in, the parameters' out
            return dict(bytes=8 * elems + 32 * pix, flops=94 * pairs)
        # parameters, both moments and the gradient out, image out, target in
        return dict(bytes=(4 + 16 + 8) * elems + (32 if case.get("alpha") else 28) * pix, flops=94 * pairs)
    if do == "warp":
        ow, oh = (int(x) for x in case["out"].split("x"))
        return dict(bytes=20 * pix + 20 * ow * oh, flops=80 * pix)
    n = case["volume"]
    if do == "seed":
        return dict(bytes=2 * n ** 3 + 56 * case["cap"], flops=20 * n ** 3)
    samples = pix * (n if do == "raymarch" else 1.0 / HIT_STEP) * _SAMPLES
    return dict(bytes=2 * n ** 3 + (16 * pix if do == "raymarch" else 60 * case["cap"]), flops=50 * samples)


# ---- the results in 64 bits ----------------------------------------------------------------

_K = dict(a=1.0925484305920792, b=0.31539156525252005, c=0.54627421529603959, d=0.59004358992664352,
          e=2.8906114426405538, f=0.45704579946446572, g=0.37317633259011540, h=1.4453057213202769)


def _basis(deg, d):
    x, y, z = d
    B = [torch.full_like(x, Y00)]
    if deg >= 1:
        B += [-0.48860251190291992 * y, 0.48860251190291992 * z, -0.48860251190291992 * x]
    if deg >= 2:
        B += [_K["a"] * x * y, -_K["a"] * y * z, _K["b"] * (2 * z * z - x * x - y * y), -_K["a"] * x * z,
              _K["c"] * (x * x - y * y)]
    if deg >= 3:
        B += [-_K["d"] * y * (3 * x * x - y * y), _K["e"] * x * y * z, -_K["f"] * y * (4 * z * z - x * x - y * y),
              _K["g"] * z * (2 * z * z - 3 * x * x - 3 * y * y), -_K["f"] * x * (4 * z * z - x * x - y * y),
              _K["h"] * z * (x * x - y * y), -_K["d"] * x * (x * x - 3 * y * y)]
    return B


def _project(P, cam, deg):
    """Screen-space splats (mean x, y, conic A, B, C, opacity, red, green, blue) of every Gaussian,
    its depth, box half sizes and whether it is drawn."""
    f64 = dict(dtype=torch.float64, device=DEV)
    W, t = torch.tensor(cam.R.astype(np.float64), **f64), torch.tensor(cam.t.astype(np.float64), **f64)
    mu, s = P[0:3], P[3:6].exp()
    w, x, y, z = P[6:10] / P[6:10].norm(dim=0, keepdim=True)
    R = [[1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)],
         [2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)],
         [2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)]]
    c = W @ mu + t[:, None]
    ok = c[2] > cam.znear
    tz = torch.where(ok, c[2], torch.ones_like(c[2]))
    rx, ry = c[0] / tz, c[1] / tz
    lx, ly = 1.3 * cam.tanx, 1.3 * cam.tany
    J = [[cam.fx / tz, -cam.fx * rx.clamp(-lx, lx) / tz], [cam.fy / tz, -cam.fy * ry.clamp(-ly, ly) / tz]]
    # rows of J W R diag(s)
    M = [[J[r][0] * W[r, k] + J[r][1] * W[2, k] for k in range(3)] for r in range(2)]
    L = [[(M[r][0] * R[0][k] + M[r][1] * R[1][k] + M[r][2] * R[2][k]) * s[k] for k in range(3)] for r in range(2)]
    sa = sum(v * v for v in L[0]) + 0.3
    sb = sum(u * v for u, v in zip(*L))
    sc = sum(v * v for v in L[1]) + 0.3
    det = sa * sc - sb * sb
    o = torch.sigmoid(P[10])
    d = mu - torch.tensor(cam.campos.astype(np.float64), **f64)[:, None]
    B = _basis(deg, d / d.norm(dim=0, keepdim=True))
    col = [sum(P[11 + 3 * k + ch] * B[k] for k in range(len(B))) + 0.5 for ch in range(3)]
    out = torch.stack([cam.fx * rx + cam.cx, cam.fy * ry + cam.cy, sc / det, -sb / det, sa / det, o,
                       *[v.clamp(min=0.0) for v in col]])
    ok = ok & (det > 0) & (o >= 1.0 / 255.0)
    k2 = 2 * (255 * o.clamp(min=1.0 / 255.0)).log()
    return out, c[2].detach(), (k2 * sa).sqrt().detach(), (k2 * sc).sqrt().detach(), ok.detach()


def _block(G, px, py):
    """Front-to-back compositing of depth-ordered splats G [9][m] over pixels (px, py): colour
    [3][p] and final transmittance [p]."""
    dx, dy = px[None, :] - G[0][:, None], py[None, :] - G[1][:, None]
    power = -0.5 * (G[2][:, None] * dx * dx + G[4][:, None] * dy * dy) - G[3][:, None] * dx * dy
    a = (G[5][:, None] * power.exp()).clamp(max=0.99)
    a = torch.where((power <= 0) & (a >= 1.0 / 255.0), a, torch.zeros_like(a))
    low = torch.log1p(-a).cumsum(0)
    a = torch.where(low >= math.log(1e-4), a, torch.zeros_like(a))   # stopped before T < 1e-4
    low = torch.log1p(-a)
    T = low.cumsum(0)
    return G[6:9] @ (a * (T - low).exp()), T[-1].exp()


def _render64(case, P, cam, bg, slope, keep):
    """Image [4][h][w] of one view in 64 bits and, where slope(image block, y0, y1, x0, x1) gives
    dL/dimage of a block of pixels, dL/dP.  keep: the pixels [h][w] composited (None: all)."""
    w, h, side = cam.width, cam.height, 64
    P = P.detach().requires_grad_(slope is not None)
    with torch.set_grad_enabled(slope is not None):
        G, depth, hx, hy, ok = _project(P, cam, case["sh"])
    g = G.detach()
    order = depth.masked_fill(~ok, math.inf).argsort(stable=True)[: int(ok.sum())]
    g, hx, hy = g[:, order].contiguous(), hx[order] + 1.0, hy[order] + 1.0
    x0, x1, y0, y1 = g[0] - hx, g[0] + hx, g[1] - hy, g[1] + hy
    img, dG, loss = torch.zeros(4, h, w, dtype=torch.float64, device=DEV), torch.zeros_like(g), 0.0
    img[:3] = bg[:, None, None]
    for by in range(0, h, side):
        rows = torch.nonzero((y1 >= by) & (y0 <= by + side)).reshape(-1)
        for bx in range(0, w, side):
            ey, ex = min(h, by + side), min(w, bx + side)
            if keep is not None and not bool(keep[by:ey, bx:ex].any()):
                continue
            at = rows[(x1[rows] >= bx) & (x0[rows] <= bx + side)]
            yy, xx = torch.meshgrid(torch.arange(by, ey, device=DEV) + 0.5, torch.arange(bx, ex, device=DEV) + 0.5,
                                    indexing="ij")
            xx, yy = xx.reshape(-1).double(), yy.reshape(-1).double()
            if at.numel():
                part = g[:, at].requires_grad_(slope is not None)
                with torch.set_grad_enabled(slope is not None):
                    C, T = _block(part, xx, yy)
                    out = torch.cat([C + T * bg[:, None], 1 - T[None]])
            else:
                part, out = None, torch.cat([bg[:, None].expand(3, xx.numel()), torch.zeros_like(xx)[None]])
            b = out.detach().reshape(4, ey - by, ex - bx)
            if keep is not None:
                b = torch.where(keep[by:ey, bx:ex], b, torch.cat([bg, bg.new_zeros(1)])[:, None, None])
            img[:, by:ey, bx:ex] = b
            if slope is not None:
                dl, add = slope(b, by, ey, bx, ex)
                loss += add
                if part is not None:
                    dG.index_add_(1, at, torch.autograd.grad(out, part, dl.reshape(4, -1))[0])
    if slope is None:
        return img, None, loss
    full = torch.zeros_like(G)
    full[:, order] = dG
    return img, torch.autograd.grad(G, P, full)[0], loss


def _random_bg(seed, views):
    """The step's background per view: SplitMix64 outputs 1 + 4 v + c, their top 24 bits."""
    out, M = np.zeros((views, 3)), (1 << 64) - 1
    for v in range(views):
        for c in range(3):
            z = (int(seed) + (1 + 4 * v + c) * 0x9E3779B97F4A7C15) & M
            z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & M
            z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & M
            out[v, c] = ((z ^ (z >> 31)) >> 40) * 2.0 ** -24
    return torch.from_numpy(out).to(DEV)


def _exact_images(case, seed):
    do, sizes = case["do"], _sizes(case)
    P, cams = _gaussians(case, seed).double(), _cameras(case, seed)
    alpha = bool(case.get("alpha"))
    bgs = _random_bg(seed, len(sizes)) if alpha else torch.zeros(len(sizes), 3, dtype=torch.float64, device=DEV)
    if do == "render":
        return torch.cat([_render64(case, P, c, bgs[v], None, None)[0].reshape(-1) for v, c in enumerate(cams)])
    keeps, tgt, off = [None] * len(sizes), None, 0
    if case.get("gaze"):   # the mask as float32 decides it, operation by operation
        for v, ((w, h), (gx, gy)) in enumerate(zip(sizes, _gaze(case, seed))):
            dx = torch.arange(w, device=DEV).float() + 0.5 - float(gx)
            dy = torch.arange(h, device=DEV).float() + 0.5 - float(gy)
            r = float(np.float32(RADIUS) * np.float32(w))
            keeps[v] = (dx * dx)[None, :] + (dy * dy)[:, None] <= float(np.float32(r) * np.float32(r))
    planes = 4 if alpha else 3
    if do == "fit":
        tgt = _targets(case, seed).double()
        count = planes * sum(int(k.sum()) if k is not None else w * h for k, (w, h) in zip(keeps, sizes))
    else:
        tgt = torch.randn(4 * sum(w * h for w, h in sizes), device=DEV, generator=_gen(seed, 8)).double()
    imgs, grads, loss = [], torch.zeros_like(P), 0.0
    for v, (w, h) in enumerate(sizes):
        if do == "fit":
            t = tgt[planes * off:planes * (off + w * h)].reshape(planes, h, w)
            if alpha:
                t = torch.cat([t[:3] + (1 - t[3:]) * bgs[v][:, None, None], t[3:]])

            def slope(b, y0, y1, x0, x1, t=t, keep=keeps[v]):
                d = b[:planes] - t[:, y0:y1, x0:x1]
                if keep is not None:
                    d = d * keep[y0:y1, x0:x1]
                dl = torch.zeros_like(b)
                dl[:planes] = d.sign() / count
                return dl, d.abs().sum() / count
        else:
            t = tgt[4 * off:4 * (off + w * h)].reshape(4, h, w)

            def slope(b, y0, y1, x0, x1, t=t):
                return t[:, y0:y1, x0:x1].contiguous(), 0.0
        img, g, add = _render64(case, P, cams[v], bgs[v], slope, keeps[v])
        imgs.append(img.reshape(-1))
        grads += g
        loss += add
        off += w * h
    if do == "autograd":
        return dict(rgba=torch.cat(imgs), grads=grads)
    # a fovea-culled step leaves the image away from the disk as it was, or as background
    return dict(loss=torch.as_tensor(loss).reshape(1), rgba=torch.cat(imgs), grads=grads,
                m=(1 - 0.9) * grads if not alpha else None, v=(1 - 0.999) * grads ** 2 if not alpha else None)


def _exact_march(case, seed):
    n, out = case["volume"], []
    vol = torch.nn.functional.pad(_volume(n, seed).double(), (1, 2, 1, 2, 1, 2)).reshape(-1)
    m, step = n + 3, float(np.float32(1.0 / n))
    lo, hi = (torch.tensor(np.array(v, np.float32).astype(np.float64), device=DEV)[:, None] for v in (TF_LO, TF_HI))
    for cam in _cameras(case, seed):
        w, h = cam.width, cam.height
        yy, xx = torch.meshgrid(torch.arange(h, device=DEV).double() + 0.5, torch.arange(w, device=DEV).double() + 0.5,
                                indexing="ij")
        d = torch.stack([(xx - cam.cx) / cam.fx, (yy - cam.cy) / cam.fy, torch.ones_like(xx)], -1).reshape(-1, 3)
        d = d @ torch.tensor(cam.R.astype(np.float64), device=DEV)
        d = (d / d.norm(dim=1, keepdim=True)).T.contiguous()
        o = torch.tensor(cam.campos.astype(np.float64), device=DEV)[:, None]
        ta, tb = (-1 - o) / d, (1 - o) / d
        t0 = torch.minimum(ta, tb).max(0).values.clamp(min=0)
        t1 = torch.maximum(ta, tb).min(0).values
        C, T = torch.zeros(3, w * h, dtype=torch.float64, device=DEV), torch.ones(w * h, dtype=torch.float64, device=DEV)
        act = torch.nonzero(t1 > t0).reshape(-1)
        k = 0
        while act.numel():
            s0 = t0[act] + k * step
            s1 = torch.minimum(s0 + step, t1[act])
            u = ((o + d[:, act] * (0.5 * (s0 + s1))) + 1) * (n / 2) - 0.5
            f0 = u.floor()
            f = u - f0
            i = (f0.long() + 1).clamp(0, m - 2)
            base = (i[0] * m + i[1]) * m + i[2]
            acc = 0.0
            for a in (0, 1):
                for b in (0, 1):
                    for c in (0, 1):
                        wt = (f[0] if a else 1 - f[0]) * (f[1] if b else 1 - f[1]) * (f[2] if c else 1 - f[2])
                        acc = acc + wt * vol[base + (a * m + b) * m + c]
            t = ((acc - THRESHOLD) / RANGE).clamp(0, 1)
            al = 1 - (-EXTINCTION * t * (s1 - s0).clamp(min=0)).exp()
            C[:, act] += (lo * (1 - t) + hi * t) * (al * T[act])
            T[act] *= 1 - al
            k += 1
            act = act[(T[act] >= T_STOP) & (t0[act] + k * step < t1[act])]
        out.append(torch.cat([C, 1 - T[None]]).reshape(-1))
    return torch.cat(out)


def _exact_seed(case, seed):
    n = case["volume"]
    vol = _volume(n, seed).reshape(-1).cpu().numpy()
    at = np.nonzero(vol > THRESHOLD)[0].astype(np.uint64)
    if at.size > case["cap"]:
        bits = np.uint64(max(1, int(n ** 3 - 1).bit_length()))
        with np.errstate(over="ignore"):
            z = np.uint64(seed) + (at + np.uint64(1)) * np.uint64(0x9E3779B97F4A7C15)
            z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
            z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
            z = z ^ (z >> np.uint64(31))
        at = np.sort(at[np.argsort(((z >> bits) << bits) | at, kind="stable")[:case["cap"]]])
    at = at.astype(np.int64)
    P = np.zeros((14, at.size))
    for a, i in enumerate((at // (n * n), at // n % n, at % n)):
        P[a] = (i + 0.5) * (2.0 / n) - 1.0
    P[3:6], P[6], P[10] = math.log(2.0 / n), 1.0, math.log(0.1 / 0.9)
    t = np.clip((vol[at] - THRESHOLD) / RANGE, 0.0, 1.0)
    for c in range(3):
        P[11 + c] = (TF_LO[c] * (1 - t) + TF_HI[c] * t - 0.5) / Y00
    return torch.from_numpy(P)


def exact(case, seed):
    do = case["do"]
    if do in ("fit", "autograd", "render"):
        got = _exact_images(case, seed)
        if case.get("gaze"):
            got["rgba"] = None   # away from the disks it holds what was there before
        return got
    if do == "raymarch":
        return _exact_march(case, seed)
    if do == "seed":
        return _exact_seed(case, seed)
    # which ray hits, and which point lands nearest on a pixel, are choices that 64 bits make
    # otherwise here and there; what follows from them is then another list
    return None
