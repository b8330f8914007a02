"""The work that users of isogs have it do, as cases to be timed.

``listed()`` names the cases, ``draw(rng)`` gives one more of the same ranges,
``prepare(case, seed)`` makes what a program holds before the call (scene, cameras,
targets, handles), ``run(state)`` is one pass through the public entry points,
``work(case)`` the bytes and operations of a pass that the path cannot do without,
and ``exact(case, seed)`` the outputs in 64 bits from plain torch, where that is quick.

Scenes are the repository's synthetic ones made on the device: isosurface points of a
sum of blobs with spectral noise (the 10k / 100k / 1M / 4M scenes) or of a perturbed
mixing layer (18M), in grid order, subsampled to the wanted count.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2509_05216_amd as P
from paper_2509_05216_amd import density, iso

DEV = "cuda"
PER_G = 11          # parameters per Gaussian besides the SH coefficients


def listed():
    return [
        # a viewer redrawing a small scene: one small image, 10k Gaussians, no SH (launches
        # and the host path count)
        dict(name="render_10k", kind="render", n=10_000, degree=0, views=1, w=256, h=256,
             tile=16, depth=256, flags=0, wide=False),
        # torch autograd user: a mini-batch of odd-sized views of a 100k scene through
        # rasterize(), a torch loss, backward
        dict(name="autograd_100k_6views", kind="autograd", n=100_000, degree=3, views=6, w=397,
             h=301, tile=16, depth=256, wide=False),
        # one training iteration of the 1M scene (splats of several pixels), statistics for
        # density control collected, as the Trainer runs it
        dict(name="train_1m_1024", kind="train", n=1_000_000, degree=3, w=1024, h=1024, tile=16,
             depth=256, collect=True, wide=True),
        # the plain step: one 2048^2 view of the 4M scene per iteration
        dict(name="train_4m_2048", kind="train", n=4_000_000, degree=3, w=2048, h=2048, tile=16,
             depth=256, collect=False, wide=False),
        # the batched step as a captured graph: 2 x 2048^2 + 2 x 1536^2 of the 4M scene
        dict(name="graph_4m_4views", kind="graph", n=4_000_000, degree=3, views=4, w=2048,
             h=2048, w2=1536, h2=1536, tile=16, depth=256, flags=3, wide=False),
        # the largest step: 18M Gaussians, two 4096^2 views
        dict(name="graph_18m_4096", kind="graph", n=18_000_000, degree=3, views=2, w=4096,
             h=4096, w2=4096, h2=4096, tile=8, depth=64, flags=0, wide=False),
        # a render server with two resident scenes and a burst of requests of mixed sizes
        dict(name="serve_burst", kind="serve", n=100_000, n2=1_000_000, requests=24, w=512,
             h=512, slots=4, batch=8),
        # the training loss and its gradient alone, three views of a size that no tile divides
        dict(name="loss_3x_1003x771", kind="loss", views=3, w=1003, h=771, grad=True),
        # the optimiser over the 4M scene
        dict(name="adam_4m", kind="adam", n=4_000_000, degree=3),
        # one densification of the 1M scene (count, then write)
        dict(name="densify_1m", kind="densify", n=1_000_000, degree=3),
        # in situ: isosurface points of a 512^3 volume ...
        dict(name="extract_512", kind="extract", nx=512, ny=512, nz=512, keep=1.0),
        # ... and ray-cast training targets of it, two 1024^2 views
        dict(name="raycast_512_1024", kind="raycast", nx=512, ny=512, nz=512, views=2, w=1024,
             h=1024),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["render", "render", "autograd", "train", "train", "graph", "graph", "serve",
                       "loss", "loss", "adam", "densify", "extract", "raycast"])
    c = dict(kind=kind)
    if kind == "render":
        tile = rng.choice([8, 16, 16, 32])
        c.update(n=_log(rng, 2_000, 2_000_000), degree=rng.choice([0, 1, 2, 3, 3]),
                 views=rng.choice([1, 1, 2, 4, 5, 8]), w=_log(rng, 64, 1400), h=_log(rng, 64, 1400),
                 tile=tile, depth=rng.choice([32, 64] if tile == 8 else [64, 128, 256]),
                 flags=rng.choice([0, 0, 1, 3]), wide=False)
    elif kind == "autograd":
        c.update(n=_log(rng, 2_000, 200_000), degree=rng.choice([0, 1, 2, 3, 3]),
                 views=rng.choice([1, 2, 3, 6]), w=_log(rng, 64, 600), h=_log(rng, 64, 600),
                 tile=rng.choice([8, 16, 16, 32]), depth=64, wide=rng.random() < 0.3)
    elif kind == "train":
        n = _log(rng, 50_000, 4_000_000)
        c.update(n=n, degree=rng.choice([0, 1, 2, 3, 3]), w=_log(rng, 256, 2048),
                 h=_log(rng, 256, 2048), tile=16, depth=256, collect=rng.random() < 0.5,
                 wide=n < 1_200_000 and rng.random() < 0.5)
    elif kind == "graph":
        n = _log(rng, 50_000, 8_000_000)
        views = rng.choice([1, 2, 4, 6, 8])
        side = lambda: _log(rng, 256, 2048 if views <= 4 else 1024)  # noqa: E731
        tile = rng.choice([8, 16, 16])
        c.update(n=n, degree=3, views=views, w=side(), h=side(), w2=side(), h2=side(), tile=tile,
                 depth=64 if tile == 8 else rng.choice([128, 256]), flags=rng.choice([0, 3, 3]),
                 wide=False)
    elif kind == "serve":
        c.update(n=_log(rng, 10_000, 300_000), n2=_log(rng, 100_000, 2_000_000),
                 requests=rng.randint(3, 32), w=_log(rng, 128, 700), h=_log(rng, 128, 700),
                 slots=rng.choice([1, 2, 4]), batch=rng.choice([1, 4, 8]))
    elif kind == "loss":
        c.update(views=rng.choice([1, 1, 2, 4]), w=_log(rng, 64, 2600), h=_log(rng, 64, 2600),
                 grad=rng.random() < 0.8)
    elif kind == "adam":
        c.update(n=_log(rng, 10_001, 4_000_000), degree=rng.choice([0, 1, 2, 3, 3]))
    elif kind == "densify":
        c.update(n=_log(rng, 20_000, 3_000_000), degree=rng.choice([0, 1, 3]))
    elif kind == "extract":
        c.update(nx=_log(rng, 48, 640), ny=_log(rng, 48, 640), nz=_log(rng, 48, 640),
                 keep=rng.choice([1.0, 1.0, 0.37]))
    else:
        c.update(nx=_log(rng, 64, 512), ny=_log(rng, 64, 512), nz=_log(rng, 64, 512),
                 views=rng.choice([1, 2, 3]), w=_log(rng, 128, 1280), h=_log(rng, 128, 1280))
    return c


# ------------------------------------------------------------------ inputs
def _gen(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1009 + salt)
    return g


def _uni(g, shape, lo, hi):
    return torch.rand(shape, generator=g, device=DEV) * (hi - lo) + lo


def _noise_terms(g, modes, kmin, kmax, amp, ax):
    """Separable factors (rows over x, y, z) of amp * sum of random cosine modes."""
    mag = torch.exp(_uni(g, (modes,), math.log(kmin), math.log(kmax)))
    d = torch.randn((modes, 3), generator=g, device=DEV)
    k = d / d.norm(dim=1, keepdim=True) * mag[:, None]
    ph = _uni(g, (modes,), 0.0, 2 * math.pi)
    a = 1.0 / mag
    a = amp * a / a.norm()
    arg = [k[:, i:i + 1] * ax[i][None, :] for i in range(3)]
    arg[2] = arg[2] + ph[:, None]
    (cx, sx), (cy, sy), (cz, sz) = [(torch.cos(t), torch.sin(t)) for t in arg]
    w = a[:, None]
    return (torch.cat([cx, sx, sx, cx]), torch.cat([cy, sy, cy, sy]),
            torch.cat([w * cz, -w * cz, -w * sz, -w * sz]))


def _blob_volume(seed, nx, ny, nz):
    """float32 (nz, ny, nx) of a blob field with spectral noise on [-1, 1]^3; level 0.5."""
    g = _gen(seed, 1)
    ax = [torch.linspace(-1, 1, m, device=DEV) for m in (nx, ny, nz)]
    nb = 96
    c = _uni(g, (nb, 3), -0.6, 0.6)
    iw = 1.0 / (2 * _uni(g, (nb, 1), 0.05, 0.17) ** 2)
    fac = [torch.exp(-((ax[i][None, :] - c[:, i:i + 1]) ** 2) * iw) for i in range(3)]
    noise = _noise_terms(g, 48, 4 * math.pi, 20 * math.pi, 0.1, ax)
    fx, fy, fz = [torch.cat([a, b]) for a, b in zip(fac, noise)]
    out = torch.empty((nz, ny, nx), device=DEV)
    for z in range(0, nz, 32):
        m = min(32, nz - z)
        rows = (fz[:, z:z + m, None] * fy[:, None, :]).reshape(fz.shape[0], m * ny)
        torch.mm(rows.t(), fx, out=out[z:z + m].view(m * ny, nx))
    return out, (-1.0, -1.0, -1.0), (1.0, 1.0, 1.0)


def _layer_volume(seed, G):
    """A thin slab of a mixing layer's volume around its interface z = -eta(x, y); level 0."""
    g = _gen(seed, 2)
    h = 2.0 / (G - 1)
    nz = int(0.3 / h)
    xs = torch.linspace(-1, 1, G, device=DEV)
    zs = (torch.arange(nz, device=DEV) - (nz - 1) / 2) * h
    eta = torch.zeros((G, G), device=DEV)
    for k in (3.0, 7.0, 15.0, 40.0, 90.0):
        a, b, p = (float(v) for v in _uni(g, (3,), -1.0, 1.0))
        eta += 0.25 / k * torch.sin(k * (a * xs[None, :] + b * xs[:, None]) + 3 * p)
    fx, fy, fz = _noise_terms(g, 16, 64 * math.pi, 256 * math.pi, 6 * h, (xs, xs, zs))
    out = torch.empty((nz, G, G), device=DEV)
    for z in range(0, nz, 16):
        m = min(16, nz - z)
        rows = (fz[:, z:z + m, None] * fy[:, None, :]).reshape(fz.shape[0], m * G)
        torch.mm(rows.t(), fx, out=out[z:z + m].view(m * G, G))
        out[z:z + m] += zs[z:z + m, None, None] + eta[None]
    half = float(zs[-1])
    return out, (-1.0, -1.0, -half), (1.0, 1.0, half)


def _crossings(vol, level, lo, hi):
    """Edge crossings (m, 3) float32 of the level in canonical (vertex, axis) order."""
    nz, ny, nx = vol.shape
    n = (nx, ny, nz)
    h = [(hi[a] - lo[a]) / (n[a] - 1) for a in range(3)]
    keys, pos = [], []
    step = max(1, (1 << 27) // (nx * ny))
    for z in range(0, nz, step):
        for a in range(3):
            end = min(nz, z + step + (1 if a == 2 else 0))
            v = vol[z:end]
            u, w = ((v[:, :, :-1], v[:, :, 1:]), (v[:, :-1], v[:, 1:]), (v[:-1], v[1:]))[a]
            at = ((u < level) != (w < level)).nonzero()
            f0, f1 = u[at[:, 0], at[:, 1], at[:, 2]], w[at[:, 0], at[:, 1], at[:, 2]]
            ok = ((f0 < level) & (f1 > level)) | ((f0 > level) & (f1 < level))
            at, f0, f1 = at[ok], f0[ok].double(), f1[ok].double()
            k = at[:, 0] + z
            keys.append(3 * ((k * ny + at[:, 1]) * nx + at[:, 2]) + a)
            p = torch.stack([lo[0] + at[:, 2].double() * h[0], lo[1] + at[:, 1].double() * h[1],
                             lo[2] + k.double() * h[2]], 1)
            p[:, a] += (f0 - level) / (f0 - f1) * h[a]
            pos.append(p)
    keys, pos = torch.cat(keys), torch.cat(pos)
    return pos[keys.argsort()], h[0]


def _scene(seed, n, degree, wide, logits=0.1):
    """Parameters of n Gaussians on an isosurface, as the framework initialises them."""
    if n > 6_000_000:
        vol, lo, hi = _layer_volume(seed, min(2048, int(math.sqrt(n) / 2.07)))
        pts, h = _crossings(vol, 0.0, lo, hi)
    else:
        G = max(24, int(math.sqrt(n) * 0.5))
        vol, lo, hi = _blob_volume(seed, G, G, G)
        pts, h = _crossings(vol, 0.5, lo, hi)
    del vol
    g = _gen(seed, 3)
    m = pts.shape[0]
    if m >= n:
        pts = pts[torch.randperm(m, generator=g, device=DEV)[:n].sort()[0]]
    else:                 # fewer crossings than wanted: repeated ones, jittered within the cell
        k = torch.randint(m, (n - m,), generator=g, device=DEV)
        more = pts[k] + (torch.rand((n - m, 3), generator=g, device=DEV).double() - 0.5) * h
        order = torch.cat([torch.arange(m, device=DEV), k]).argsort(stable=True)
        pts = torch.cat([pts, more])[order]
    rows = (degree + 1) ** 2 * 3
    ls = _uni(g, (3, n), -5.0, -3.0) if wide else math.log(h) + _uni(g, (3, n), -0.5, 0.5)
    q = torch.randn((4, n), generator=g, device=DEV)
    op = torch.full((n,), 0.1, device=DEV) if logits == 0.1 else _uni(g, (n,), 0.0, 4.0)
    sh = torch.randn((rows, n), generator=g, device=DEV) * 0.1
    return P.Params(pts.t().float().contiguous(), ls.contiguous(), q / q.norm(dim=0, keepdim=True),
                    op, sh, degree)


def _cams(sizes, seed):
    """Cameras of the orbit, one per (w, h), starting at a seeded place on it."""
    out = []
    for i, (w, h) in enumerate(sizes):
        out.append(P.orbit_cameras(64, 2.5, 60.0, w, h)[(7 * int(seed) + 23 * i + 11) % 64])
    return out


def _target(g, w, h):
    """A shaded, textured object on black, (3, h, w)."""
    y, x = torch.meshgrid(torch.linspace(-1, 1, h, device=DEV), torch.linspace(-1, 1, w, device=DEV),
                          indexing="ij")
    k = _uni(g, (6,), 3.0, 40.0).tolist()
    r2 = x * x + y * y + 0.2 * torch.sin(k[0] * x) * torch.sin(k[1] * y)
    lit = torch.sqrt(torch.clamp(0.7 - r2, min=0.0))
    tex = [0.6 + 0.25 * torch.sin(k[i] * x + k[5 - i] * y + i) for i in range(3)]
    return torch.stack([lit * t for t in tex]).contiguous()


def _sizes(c):
    if "w2" in c:
        half = (c["views"] + 1) // 2
        return [(c["w"], c["h"])] * half + [(c["w2"], c["h2"])] * (c["views"] - half)
    return [(c["w"], c["h"])] * c.get("views", 1)


_ctx = {}


def _context():
    """One library context per process, as a program keeps it."""
    if "c" not in _ctx:
        _ctx["c"] = P.Context(torch.cuda.current_device())
    return _ctx["c"]


def _training_state(seed, n, degree):
    """Parameters, gradients and Adam moments in the middle of a training run."""
    g = _gen(seed, 5)
    p = P.Params(_uni(g, (3, n), -1, 1), _uni(g, (3, n), -6, -3),
                 torch.randn((4, n), generator=g, device=DEV), _uni(g, (n,), -3, 3),
                 torch.randn(((degree + 1) ** 2 * 3, n), generator=g, device=DEV) * 0.1, degree)
    like = lambda f: P.Params(*(f(t) for t in p.tensors()), degree)  # noqa: E731
    grad = like(lambda t: torch.randn(t.shape, generator=g, device=DEV) * 1e-4)
    m = like(lambda t: torch.randn(t.shape, generator=g, device=DEV) * 3e-5)
    v = like(lambda t: torch.rand(t.shape, generator=g, device=DEV) * 1e-8 + 1e-12)
    return p, grad, m, v


def _densify_inputs(c, seed):
    n, deg = c["n"], c["degree"]
    p, _, m, v = _training_state(seed, n, deg)
    # statistics of an interval: about a tenth selected, clones and splits, some to prune;
    # what decides is the same for every seed, so that the output sizes are
    g = _gen(0, 6)
    p.log_scales.copy_(_uni(g, (3, n), -6, -3))
    stats = density.DensityStats(
        torch.rand((n,), generator=g, device=DEV) ** 4 * 3e-3,
        torch.randint(0, 12, (n,), generator=g, device=DEV, dtype=torch.int32),
        torch.randint(0, 30, (n,), generator=g, device=DEV, dtype=torch.int32))
    p.opacity_logits.copy_(_uni(g, (n,), -6.5, 3.0))
    return p, m, v, stats


def prepare(c, seed):
    ctx, kind = _context(), c["kind"]
    s = dict(kind=kind, ctx=ctx, case=c)
    g = _gen(seed, 4)
    if kind in ("render", "autograd", "train", "graph"):
        s["p"] = _scene(seed, c["n"], c["degree"], c["wide"], 1.0 if kind == "render" else 0.1)
        s["cams"] = _cams(_sizes(c), seed)
    if kind == "render":
        s["frame"] = P.Frame()
        s["images"] = [torch.empty((3, k.height, k.width), device=DEV) for k in s["cams"]]
    elif kind == "autograd":
        s["leaves"] = [t.requires_grad_(True) for t in s["p"].tensors()]
        s["target"] = torch.stack([_target(g, *z) for z in _sizes(c)])
    elif kind == "train":
        cam = s["cams"][0]
        s["frame"] = P.Frame()
        s["target"] = _target(g, cam.width, cam.height)
        s["image"], s["dl"] = torch.empty_like(s["target"]), torch.empty_like(s["target"])
        s["loss"], s["grads"] = torch.zeros(1, device=DEV), s["p"].zeros_like()
        s["stats"] = density.DensityStats.zeros(c["n"], DEV) if c["collect"] else None
    elif kind == "graph":
        targets = [_target(g, *z) for z in _sizes(c)]
        s["graph"] = P.StepGraph(ctx, s["p"], s["cams"], targets, with_adam=False, render=dict(
            tile=c["tile"], lds_depth=c["depth"], flags=c["flags"]))
    elif kind == "serve":
        s["server"] = P.Server(ctx, n_slots=c["slots"], max_batch_views=c["batch"])
        s["scenes"] = [_scene(seed, c["n"], 3, False, 1.0), _scene(seed + 1, c["n2"], 3, False, 1.0)]
        ids = [s["server"].add_scene(p) for p in s["scenes"]]
        sizes = [(k * c["w"], k * c["h"]) for k in (1, 2)]
        s["requests"] = []
        for i in range(c["requests"]):
            w, h = sizes[1 if i % 4 == 3 else 0]
            cam = _cams([(w, h)], seed + 5 * i)[0]
            s["requests"].append((ids[i % 2], i % 2, cam, torch.empty((3, h, w), device=DEV)))
    elif kind == "loss":
        s["cams"] = _cams(_sizes(c), seed)
        s["y"] = [_target(g, *z) for z in _sizes(c)]
        s["x"] = [(t + 0.05 * torch.randn(t.shape, generator=g, device=DEV) * (t > 0)).clamp(0, 1)
                  for t in s["y"]]
    elif kind == "adam":
        s["p"], s["g"], s["m"], s["v"] = _training_state(seed, c["n"], c["degree"])
        s["step"] = 200
    elif kind == "densify":
        s["p"], s["m"], s["v"], s["stats"] = _densify_inputs(c, seed)
        s["seed"] = int(seed)
    elif kind in ("extract", "raycast"):
        vol, lo, hi = _blob_volume(seed if kind == "raycast" else 0, c["nx"], c["ny"], c["nz"])
        s["vol"] = iso.Volume(vol, lo, hi)
        if kind == "extract":
            # the same crossed edges for every seed (the number of points is), other values
            for z in range(0, c["nz"], 64):
                part = vol[z:z + 64]
                part.sub_(0.5).mul_(_uni(g, part.shape, 0.8, 1.25)).add_(0.5)
        else:
            s["cams"] = _cams(_sizes(c), seed)
            s["step"] = 2.0 / (max(c["nx"], c["ny"], c["nz"]) - 1)
    return s


# ------------------------------------------------------------------ the calls
def run(s):
    kind, ctx, c = s["kind"], s["ctx"], s["case"]
    if kind == "render":
        P.render_fwd(ctx, s["p"], s["cams"], s["images"], tile=c["tile"], lds_depth=c["depth"],
                     flags=c["flags"], frame=s["frame"])
        return s["images"]
    if kind == "autograd":
        for t in s["leaves"]:
            t.grad = None
        img = P.rasterize(ctx, s["leaves"], c["degree"], s["cams"], tile=c["tile"],
                          lds_depth=c["depth"])
        loss = ((img - s["target"]) ** 2).mean()
        loss.backward()
        return [img.detach(), loss.detach()] + [t.grad for t in s["leaves"]]
    if kind == "train":
        P.render_fwd(ctx, s["p"], s["cams"], [s["image"]], tile=c["tile"], lds_depth=c["depth"],
                     flags=4 if c["collect"] else 0, frame=s["frame"])
        P.loss_grad_into(ctx, [s["image"]], [s["target"]], s["cams"], s["loss"], [s["dl"]])
        P.render_bwd(ctx, s["frame"], s["p"], [s["dl"]], s["grads"], keep_screen=c["collect"])
        out = [s["image"], s["loss"], *s["grads"].tensors()]
        if c["collect"]:
            density.accumulate(ctx, s["frame"], s["stats"])
            out += [s["stats"].grad, s["stats"].count, s["stats"].max_radius]
        return out
    if kind == "graph":
        g = s["graph"]
        g.launch()
        return [g.images, g.loss, g.grads.tensors()]
    if kind == "serve":
        for sid, _, cam, out in s["requests"]:
            s["server"].submit(sid, cam, out)
        s["server"].drain()
        return [r[3] for r in s["requests"]]
    if kind == "loss":
        if c["grad"]:
            return P.loss_grad(ctx, s["x"], s["y"], s["cams"])
        return P.core.image_metrics(ctx, s["x"], s["y"], s["cams"])
    if kind == "adam":
        s["step"] += 1
        P.adam_step(ctx, s["p"], s["g"], s["m"], s["v"], s["step"])
        return [t for q in (s["p"], s["m"], s["v"]) for t in q.tensors()]
    if kind == "densify":
        p, m, v, info, src = density.densify(ctx, s["p"], s["m"], s["v"], s["stats"], 2.5,
                                             seed=s["seed"], max_screen=20.0, want_src=True)
        return [[t for q in (p, m, v) for t in q.tensors()], info, src]
    if kind == "extract":
        return iso.extract(ctx, s["vol"], 0.5, c["keep"], 7)
    return iso.raycast(ctx, s["vol"], s["cams"], 0.5, s["step"])


# ------------------------------------------------------------------ what a pass cannot do without
def work(c):
    """Compulsory bytes (inputs read once, outputs written once) and operations.  The
    rendering operations depend on the image content; a typical 100 (pixel, Gaussian)
    pairs per pixel at 20 (forward) or 70 (forward and backward) each stand for them."""
    kind = c["kind"]
    if kind in ("render", "autograd", "train", "graph"):
        n, pix = c["n"], sum(w * h for w, h in _sizes(c))
        par = 4 * (PER_G + (c["degree"] + 1) ** 2 * 3) * n
        if kind == "render":
            return dict(bytes=par + 12 * pix, flops=2000 * pix)
        extra = (20 if kind == "train" and c["collect"] else 0) * n
        return dict(bytes=2 * par + 36 * pix + extra, flops=7000 * pix + 400 * pix)
    if kind == "serve":
        px = c["w"] * c["h"]
        pix = sum(px * (4 if i % 4 == 3 else 1) for i in range(c["requests"]))
        return dict(bytes=4 * 59 * (c["n"] + c["n2"]) + 12 * pix, flops=2000 * pix)
    if kind == "loss":
        pix = c["views"] * c["w"] * c["h"]
        return dict(bytes=(36 if c["grad"] else 24) * pix, flops=(1000 if c["grad"] else 600) * pix)
    if kind == "adam":
        k = (PER_G + (c["degree"] + 1) ** 2 * 3) * c["n"]
        return dict(bytes=28 * k, flops=14 * k)
    if kind == "densify":
        k = (PER_G + (c["degree"] + 1) ** 2 * 3) * c["n"]
        return dict(bytes=24 * k + 12 * c["n"], flops=40 * c["n"])
    vox = c["nx"] * c["ny"] * c["nz"]
    if kind == "extract":
        side = (c["nx"] * c["ny"] + c["ny"] * c["nz"] + c["nx"] * c["nz"]) / 3
        return dict(bytes=4 * vox + 48 * side * c["keep"], flops=6 * vox)
    pix = c["views"] * c["w"] * c["h"]
    steps = max(c["nx"], c["ny"], c["nz"]) * 0.5
    return dict(bytes=4 * vox + 12 * pix, flops=30 * steps * pix)


# ------------------------------------------------------------------ 64-bit references
def exact(c, seed):
    kind = c["kind"]
    if kind in ("train", "graph"):
        return None          # minutes in plain torch
    if kind in ("render", "autograd", "serve"):
        return _exact_render(c, seed)
    s = prepare(c, seed)
    if kind == "loss":
        return _exact_loss(s)
    if kind == "adam":
        return _exact_adam(s)
    if kind == "densify":
        return _exact_densify(s)
    if kind == "extract":
        return _exact_extract(s)
    return _exact_raycast(s)


def _exact_adam(s):
    step, lr = s["step"] + 1, P.core.DEFAULT_LR
    f32 = lambda v: float(np.float32(v))  # noqa: E731
    b1, b2, eps = f32(0.9), f32(0.999), f32(1e-15)
    outs = [[], [], []]
    for name, p, g, m, v in zip(P.core.PARAM_KEYS, *(s[k].tensors() for k in "pgmv")):
        p, g, m, v = (t.double() for t in (p, g, m, v))
        m = b1 * m + (1 - b1) * g
        v = b2 * v + (1 - b2) * g * g
        up = (m / (1 - b1 ** step)) / ((v / (1 - b2 ** step)).sqrt() + eps)
        if name == "sh":
            rate = torch.full((p.shape[0], 1), f32(lr["sh_rest"]), device=DEV, dtype=torch.float64)
            rate[:3] = f32(lr["sh_dc"])
        else:
            rate = f32(lr[name])
        for o, t in zip(outs, (p - rate * up, m, v)):
            o.append(t)
    return [t for o in outs for t in o]


def _window():
    w = torch.exp(-torch.arange(-5, 6, device=DEV, dtype=torch.float64) ** 2 / 4.5)
    return w / w.sum()


def _blur(t):
    """Separable 11-tap window with zero padding over the last two axes."""
    w = _window()
    for dim in (-1, -2):
        pad = (5, 5, 0, 0) if dim == -1 else (0, 0, 5, 5)
        q, n = torch.nn.functional.pad(t, pad), t.shape[dim]
        t = sum(w[i] * q.narrow(dim, i, n) for i in range(11))
    return t


def _exact_loss(s):
    lam, nv = 0.2, len(s["x"])
    total, grads, rows = 0.0, [], []
    for x, y in zip(s["x"], s["y"]):
        x, y = x.double(), y.double()
        mx, my = _blur(x), _blur(y)
        sxx, syy, sxy = _blur(x * x) - mx * mx, _blur(y * y) - my * my, _blur(x * y) - mx * my
        a1, a2 = 2 * mx * my + 1e-4, 2 * sxy + 9e-4
        b1, b2 = mx * mx + my * my + 1e-4, sxx + syy + 9e-4
        S = a1 * a2 / (b1 * b2)
        g1 = 2 * (my * (a2 - a1) / (b1 * b2) + S * mx * (1 / b2 - 1 / b1))
        g2, g3 = -S / b2, 2 * a1 / (b1 * b2)
        l1 = (x - y).abs().mean()
        total = total + (1 - lam) * l1 + lam * (1 - S.mean())
        ds = _blur(g1) + 2 * x * _blur(g2) + y * _blur(g3)
        grads.append(((1 - lam) * torch.sign(x - y) - lam * ds) / (x.numel() * nv))
        mse = ((x - y) ** 2).mean()
        rows.append(torch.stack([mse, -10 * torch.log10(mse), l1, S.mean()]))
    if s["case"]["grad"]:
        return (total / nv).reshape(1), grads
    return torch.stack(rows)


def _philox(ctr, k0, k1):
    """Philox4x32-10 on int64 tensors holding 32-bit words."""
    mask = 0xFFFFFFFF

    def mul(a, b):           # high and low words of a 32 x 32 bit product
        lo = a * (b & 0xFFFF)
        hi = a * (b >> 16) + (lo >> 16)
        return hi >> 16, ((hi << 16) | (lo & 0xFFFF)) & mask

    c = list(ctr)
    for _ in range(10):
        h0, l0 = mul(c[0], 0xD2511F53)
        h1, l1 = mul(c[2], 0xCD9E8D57)
        c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    return c


def _exact_densify(s):
    p, st, n = s["p"], s["stats"], s["case"]["n"]
    ext, div = 2.5, 1.6
    g = torch.where(st.count > 0, st.grad.double() / st.count.clamp(min=1).double(),
                    torch.zeros((), device=DEV, dtype=torch.float64))
    sel = g >= 0.0002
    ls = p.log_scales.double()
    smax = torch.exp(ls).amax(0)
    cmax = torch.exp(ls - math.log(div)).amax(0)
    low = torch.sigmoid(p.opacity_logits.double()) < 0.005
    big = smax > 0.1 * ext
    clone, split = sel & (smax <= 0.01 * ext), sel & (smax > 0.01 * ext)
    keep = ~split & ~low & ~((st.max_radius > 20) | big)
    made = clone & ~low & ~big
    child = split & ~low & ~(cmax > 0.1 * ext)
    ik, ic, iw = (t.nonzero()[:, 0] for t in (keep, made, child))
    iw2 = iw.repeat_interleave(2)
    src = torch.cat([ik, ic, iw2])
    ch = torch.arange(2, device=DEV).repeat(iw.shape[0])
    one = torch.zeros_like(iw2)
    c = _philox([iw2, 16 + ch, one, one], s["seed"] & 0xFFFFFFFF, s["seed"] >> 32)

    def normals(a, b):
        u = ((a >> 8).double() + 0.5) * 2.0 ** -24
        r, th = torch.sqrt(-2 * torch.log(u)), 2 * math.pi * ((b >> 8).double() * 2.0 ** -24)
        return r * torch.cos(th), r * torch.sin(th)

    z = torch.stack([*normals(c[0], c[1]), normals(c[2], c[3])[0]])
    off = _matvec(_rotation(p.quats.double()[:, iw2]), torch.exp(ls[:, iw2]) * z)
    outs = []
    new = torch.arange(src.shape[0], device=DEV) >= ik.shape[0]
    drawn = torch.arange(src.shape[0], device=DEV) >= ik.shape[0] + ic.shape[0]
    for name, t in zip(P.core.PARAM_KEYS, p.tensors()):
        o = t[..., src].double()
        if name == "means":
            o[:, drawn] += off
        elif name == "log_scales":
            o[:, drawn] -= math.log(div)
        outs.append(o)
    for q in (s["m"], s["v"]):
        for t in q.tensors():
            o = t[..., src].double()
            o[..., new] = 0
            outs.append(o)
    return [outs, None, None]


def _exact_extract(s):
    v, c = s["vol"], s["case"]
    if c["keep"] < 1.0:      # which crossings stay is a random draw of the library's
        return None
    return _crossings(v.values, 0.5, v.lo, v.hi)[0].t()


def _exact_raycast(s):
    vol, out = s["vol"], []
    val = vol.values.reshape(-1)
    nz, ny, nx = vol.values.shape
    n = torch.tensor([nx, ny, nz], device=DEV)
    f64 = dict(device=DEV, dtype=torch.float64)
    lo, hi = torch.tensor(vol.lo, **f64), torch.tensor(vol.hi, **f64)
    h = (hi - lo) / (n - 1)
    step = float(np.float32(s["step"]))

    def trilerp(p, want_grad=False):
        u = (p - lo) / h
        i = torch.minimum(u.floor().long().clamp(min=0), n - 2)
        fx, fy, fz = (u - i).unbind(1)
        b = (i[:, 2] * ny + i[:, 1]) * nx + i[:, 0]
        v = [val[b + dz * ny * nx + dy * nx + dx].double()
             for dz in (0, 1) for dy in (0, 1) for dx in (0, 1)]
        x = [v[2 * k] + fx * (v[2 * k + 1] - v[2 * k]) for k in range(4)]
        y = [x[0] + fy * (x[1] - x[0]), x[2] + fy * (x[3] - x[2])]
        f = y[0] + fz * (y[1] - y[0])
        if not want_grad:
            return f
        d = [v[2 * k + 1] - v[2 * k] for k in range(4)]
        gx = (d[0] * (1 - fy) + d[1] * fy) * (1 - fz) + (d[2] * (1 - fy) + d[3] * fy) * fz
        gy = (x[1] - x[0]) * (1 - fz) + (x[3] - x[2]) * fz
        return torch.stack([gx, gy, y[1] - y[0]], 1) / h

    for cam in s["cams"]:
        k = P.camera_to_dict(cam)
        R, t = torch.tensor(k["R"], **f64), torch.tensor(k["t"], **f64)
        W, H = k["width"], k["height"]
        y, x = torch.meshgrid(torch.arange(H, **f64), torch.arange(W, **f64), indexing="ij")
        d = torch.stack([(x.reshape(-1) + 0.5 - k["cx"]) / k["fx"],
                         (y.reshape(-1) + 0.5 - k["cy"]) / k["fy"], torch.ones(W * H, **f64)], 1) @ R
        d = d / d.norm(dim=1, keepdim=True)
        o = -(R.t() @ t)
        t0, t1 = (lo - o) / d, (hi - o) / d
        tn = torch.minimum(t0, t1).amax(1).clamp(min=0)
        tf = torch.maximum(t0, t1).amin(1)
        live = (tf > tn).nonzero()[:, 0]
        hit_t = torch.full((W * H,), -1.0, **f64)
        fp = trilerp(o + tn[live, None] * d[live]) - 0.5
        j = 0
        while live.numel():
            j += 1
            tk = tn[live] + j * step
            f = trilerp(o + tk[:, None] * d[live]) - 0.5
            inside = tk <= tf[live]
            rise = inside & (fp < 0) & (f >= 0)
            hit_t[live[rise]] = tk[rise]
            go = inside & ~rise
            live, fp = live[go], f[go]
        at = (hit_t >= 0).nonzero()[:, 0]
        b = hit_t[at]
        a = b - step
        dd = d[at]
        for _ in range(10):
            mid = 0.5 * (a + b)
            below = trilerp(o + mid[:, None] * dd) - 0.5 < 0
            a, b = torch.where(below, mid, a), torch.where(below, b, mid)
        q = o + (0.5 * (a + b))[:, None] * dd
        gr = trilerp(q, True)
        lam = ((gr * dd).sum(1) / gr.norm(dim=1)).abs()
        sh = 0.2 + 0.8 * lam
        img = torch.zeros((3, W * H), **f64)
        img[:, at] = torch.stack([0.85 * sh, (0.45 + 0.25 * q[:, 2]) * sh,
                                  (0.30 + 0.25 * (q[:, 0] + 1)) * sh])
        out.append(img.view(3, H, W))
    return out


def _rotation(q):
    w, x, y, z = q / q.norm(dim=0, keepdim=True)
    return ((1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)),
            (2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)),
            (2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)))


def _matvec(R, v):
    return torch.stack([R[r][0] * v[0] + R[r][1] * v[1] + R[r][2] * v[2] for r in range(3)])


def _sh(x, y, z, degree):
    """Real SH basis, Condon-Shortley phase, m = -l..l."""
    pi = math.pi
    one = torch.ones_like(x)
    Y = [math.sqrt(1 / (4 * pi)) * one]
    if degree > 0:
        k = math.sqrt(3 / (4 * pi))
        Y += [-k * y, k * z, -k * x]
    if degree > 1:
        k = math.sqrt(15 / pi) / 2
        Y += [k * x * y, -k * y * z, math.sqrt(5 / pi) / 4 * (2 * z * z - x * x - y * y), -k * x * z,
              k / 2 * (x * x - y * y)]
    if degree > 2:
        a, b, c = (math.sqrt(35 / (2 * pi)) / 4, math.sqrt(105 / pi) / 2, math.sqrt(21 / (2 * pi)) / 4)
        e = math.sqrt(7 / pi) / 4
        Y += [-a * y * (3 * x * x - y * y), b * x * y * z, -c * y * (4 * z * z - x * x - y * y),
              e * z * (2 * z * z - 3 * x * x - 3 * y * y), -c * x * (4 * z * z - x * x - y * y),
              b / 2 * z * (x * x - y * y), -a * x * (x * x - 3 * y * y)]
    return Y


def _project(p, degree, k):
    """Screen-space (9, n): mean, conic, opacity, rgb; rectangle of pixels, depth, touched."""
    mu, ls, q, logit, sh = p
    f64 = dict(device=DEV, dtype=torch.float64)
    R, t = torch.tensor(k["R"], **f64), torch.tensor(k["t"], **f64)
    W, H, fx, fy = k["width"], k["height"], k["fx"], k["fy"]
    tc = R @ mu + t[:, None]
    vis = tc[2] > k["z_near"]
    tz = torch.where(vis, tc[2], torch.ones_like(tc[2]))
    xz, yz = tc[0] / tz, tc[1] / tz
    lx, ly = 1.3 * 0.5 * W / fx, 1.3 * 0.5 * H / fy
    u, v = xz.clamp(-lx, lx), yz.clamp(-ly, ly)
    Rq = _rotation(q)
    s = torch.exp(ls)
    M = [[Rq[r][c] * s[c] for c in range(3)] for r in range(3)]
    T0 = [fx / tz * R[0, j] - fx * u / tz * R[2, j] for j in range(3)]
    T1 = [fy / tz * R[1, j] - fy * v / tz * R[2, j] for j in range(3)]
    A0 = [sum(T0[r] * M[r][c] for r in range(3)) for c in range(3)]
    A1 = [sum(T1[r] * M[r][c] for r in range(3)) for c in range(3)]
    a = sum(x * x for x in A0) + 0.3
    b = sum(x * y for x, y in zip(A0, A1))
    c = sum(x * x for x in A1) + 0.3
    det = a * c - b * b
    mx, my = fx * xz + k["cx"], fy * yz + k["cy"]
    d = mu - (-(R.t() @ t))[:, None]
    d = d / d.norm(dim=0, keepdim=True)
    Y = torch.stack(_sh(d[0], d[1], d[2], degree))
    rgb = ((sh.view(Y.shape[0], 3, -1) * Y[:, None]).sum(0) + 0.5).clamp(min=0)
    scr = torch.cat([torch.stack([mx, my, c / det, -b / det, a / det, torch.sigmoid(logit)]), rgb])
    with torch.no_grad():
        lmax = 0.5 * (a + c) + torch.sqrt((0.5 * (a - c)) ** 2 + b * b)
        r = torch.ceil(3 * torch.sqrt(lmax))
        x0, x1 = torch.ceil(mx - 0.5 - r).clamp(min=0), torch.floor(mx - 0.5 + r).clamp(max=W - 1)
        y0, y1 = torch.ceil(my - 0.5 - r).clamp(min=0), torch.floor(my - 0.5 + r).clamp(max=H - 1)
        touched = vis & (x0 <= x1) & (y0 <= y1)
    return scr, (x0, y0, x1, y1), tc[2].detach().float(), touched


def _tile(s, X, Y):
    """Colours (3, pixels) of one tile's ordered splats s (9, L)."""
    dx, dy = X[:, None] - s[0], Y[:, None] - s[1]
    power = -0.5 * (s[2] * dx * dx + s[4] * dy * dy) - s[3] * dx * dy
    alpha = (s[5] * torch.exp(power)).clamp(max=0.99)
    alpha = alpha * ((power <= 0) & (alpha >= 1 / 255))
    lt = torch.log1p(-alpha).cumsum(1)
    before = torch.exp(lt - torch.log1p(-alpha))
    w = alpha * before * (torch.exp(lt) >= 1e-4)
    return (s[6:9, None, :] * w).sum(2)


def _exact_view(p, degree, cam, tile, image, dl=None):
    """Composites one view into `image`; with dl, backpropagates it into the leaves p."""
    k = P.camera_to_dict(cam)
    W, H = k["width"], k["height"]
    scr, (x0, y0, x1, y1), depth, touched = _project(p, degree, k)
    order = torch.argsort(depth, stable=True)
    order = order[touched[order]]
    box = [(t[order] // tile).long() for t in (x0, y0, x1, y1)]
    flat = scr.detach()[:, order]
    gs = torch.zeros_like(flat)
    for ty in range(-(-H // tile)):
        row = ((box[1] <= ty) & (box[3] >= ty)).nonzero()[:, 0]
        rx0, rx1 = box[0][row], box[2][row]
        for tx in range(-(-W // tile)):
            at = row[(rx0 <= tx) & (rx1 >= tx)]
            if at.numel() == 0:
                continue
            ys, xs = slice(ty * tile, min(H, ty * tile + tile)), slice(tx * tile, min(W, tx * tile + tile))
            Y, X = torch.meshgrid(torch.arange(ys.start, ys.stop, device=DEV, dtype=torch.float64) + 0.5,
                                  torch.arange(xs.start, xs.stop, device=DEV, dtype=torch.float64) + 0.5,
                                  indexing="ij")
            s = flat[:, at].requires_grad_(dl is not None)
            out = _tile(s, X.reshape(-1), Y.reshape(-1))
            image[:, ys, xs] = out.detach().view(3, *X.shape)
            if dl is not None:
                gs[:, at] += torch.autograd.grad(out, s, dl[:, ys, xs].reshape(3, -1))[0]
    if dl is not None:
        full = torch.zeros_like(scr)
        full[:, order] = gs
        scr.backward(full)


def _exact_render(c, seed):
    s = prepare(c, seed)
    if c["kind"] == "serve":
        jobs = [(s["scenes"][k], cam, 16) for _, k, cam, _ in s["requests"]]
    else:
        jobs = [(s["p"], cam, c["tile"]) for cam in s["cams"]]
    tiles = sum((cam.width // 16 + 1) * (cam.height // 16 + 1) for _, cam, _ in jobs)
    if c.get("wide"):
        tiles *= 3
    both = c["kind"] == "autograd"
    if tiles * (3 if both else 1) > 12_000:      # over about 20 seconds
        return None
    images, leaves = [], None
    for p, cam, tile in jobs:
        image = torch.zeros((3, cam.height, cam.width), device=DEV, dtype=torch.float64)
        p64 = [t.detach().double() for t in p.tensors()]
        with torch.no_grad():
            _exact_view(p64, p.sh_degree, cam, tile, image)
        images.append(image)
    if not both:
        return images
    img, target = torch.stack(images), s["target"].double()
    dl = 2 * (img - target) / img.numel()
    leaves = [t.detach().double().requires_grad_(True) for t in s["p"].tensors()]
    for v, cam in enumerate(s["cams"]):
        _exact_view(leaves, c["degree"], cam, c["tile"], torch.empty_like(images[v]), dl[v])
    return [img, ((img - target) ** 2).mean()] + [t.grad for t in leaves]
