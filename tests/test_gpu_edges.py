"""Kernels at the sizes where their tiling can go wrong (block edges, remainders, list
capacities), against the float64 oracle."""
import numpy as np
import pytest
import torch

from tests._parity import rel_l2
from tests.test_gpu_density import _check_densify

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2509_05216_amd as P
    return P


@pytest.fixture(scope="module")
def ctx(P):
    return P.Context(0)


# ---------------------------------------------------------------- densify
@pytest.mark.parametrize("n,deg,n_split", [
    (1024, 3, 8),      # one block, far more outputs than one run of it holds
    (2049, 0, 8),      # the fewest rows, a one-Gaussian last block
    (5000, 1, 5)])
def test_densify_many_children(P, ctx, n, deg, n_split):
    from paper_2509_05216_amd import density as D
    ri = _check_densify(P, D, ctx, n, deg, 31 + n, 20.0, n_split)
    assert ri["children"] > 0


# ---------------------------------------------------------------- extraction
def _volume(kind, shape):
    nx, ny, nz = shape
    z, y, x = np.meshgrid(*(np.linspace(-1, 1, m) for m in (nz, ny, nx)), indexing="ij")
    if kind == "sphere":
        return (1.1 - np.sqrt(x * x + y * y + z * z)).astype(np.float32)
    v = np.random.default_rng(nx).random((nz, ny, nx)).astype(np.float32)
    if kind == "checker":   # every edge of the grid crosses
        i, j, k = np.meshgrid(*(np.arange(m) for m in (nz, ny, nx)), indexing="ij")
        return np.where((i + j + k) % 2 == 0, 0.2, 0.9).astype(np.float32) + 0.05 * v
    if kind == "ties":      # values on the level (never a crossing), NaN and infinities
        v = np.round(v * 4) / 4
        v.reshape(-1)[::7] = np.nan
        v.reshape(-1)[3::11] = np.inf
        v.reshape(-1)[5::13] = -np.inf
    return v.astype(np.float32)


@pytest.mark.parametrize("kind,shape,keep", [
    ("noise", (2, 3, 5000), 1.0), ("noise", (3, 5, 4), 0.5), ("noise", (4099, 3, 3), 1.0),
    ("noise", (2, 2049, 2), 1.0), ("checker", (33, 31, 29), 1.0), ("checker", (64, 64, 4), 0.25),
    ("ties", (40, 41, 13), 1.0),
    ("sphere", (263, 256, 257), 1.0)])    # more than 4096 blocks of 4096 vertices
def test_extraction_block_edges(P, ctx, kind, shape, keep):
    from oracle import iso as OI
    from paper_2509_05216_amd import iso
    vol = _volume(kind, shape)
    lo, hi = (-1.0, -1.0, -1.0), (1.0, 1.0, 1.0)
    got = iso.extract(ctx, iso.Volume(torch.tensor(vol, device="cuda"), lo, hi), 0.5, keep, 9)
    got = got.cpu().numpy()
    with np.errstate(invalid="ignore"):
        want, m = OI.extract(vol, lo, hi, 0.5, keep, 9)
    assert m > 0 and got.shape == want.shape
    # float64 positions rounded once: within one float32 ulp
    both = np.isfinite(want)
    assert np.array_equal(both, np.isfinite(got))
    ulp = np.spacing(np.abs(want[both]).astype(np.float32)).astype(np.float64)
    assert np.all(np.abs(got[both].astype(np.float64) - want[both]) <= ulp)


def _ray_volume(kind, shape, rng):
    """float32 (nz, ny, nx) around the level 0.5 (or 0 for "zero")."""
    nz, ny, nx = shape
    z, y, x = np.meshgrid(*(np.linspace(-1, 1, k) for k in shape), indexing="ij")
    if kind == "shell":              # long one-sided runs, then a thin wall
        v = 0.5 + 0.4 * np.cos(9 * x) - 0.3 * y * z - 0.25
    elif kind == "noise":            # a crossing in most cells
        v = rng.random(shape)
    elif kind == "ties":             # samples that equal the level exactly
        v = rng.integers(0, 3, shape) * 0.25 + 0.25
    elif kind == "zero":             # level 0, values of very different size
        v = (x + 0.1 * y) * 10.0 ** (6 * z)
    else:                            # not finite in places
        v = 0.5 + 0.4 * np.cos(7 * x)
        v[nz // 2, ny // 2, nx // 3] = np.nan
        v[nz // 3, ny // 2, nx // 2] = np.inf
        v[0, ny // 2, (2 * nx) // 3] = -np.inf
    return v.astype(np.float32)


@pytest.mark.parametrize("kind,shape,step", [
    ("shell", (5, 6, 421), 0.006), ("shell", (390, 4, 9), 0.0051), ("shell", (2, 401, 5), 0.004),
    ("noise", (6, 7, 400), 0.005), ("ties", (7, 395, 6), 0.005), ("zero", (5, 8, 403), 0.0055),
    ("odd", (6, 9, 400), 0.005), ("shell", (17, 16, 18), 0.11), ("ties", (9, 8, 7), 0.05),
    ("odd", (12, 11, 13), 0.07), ("zero", (2, 2, 2), 0.03),
])
def test_raycast_routes_match_oracle(P, kind, shape, step):
    """Rays through cell classes (long volumes) and without them (small ones), from
    outside and inside the box, along an axis, and at one-sided, level-valued and
    non-finite samples: the float64 oracle's image, to the rounding of a float32 image."""
    from oracle import camera as ocam
    from oracle import iso as OI
    from paper_2509_05216_amd import iso
    rng = np.random.default_rng(7)
    vol = _ray_volume(kind, shape, rng)
    level = 0.0 if kind == "zero" else 0.5
    step = float(np.float32(step))
    cams = [ocam.to_float32(c) for c in ocam.orbit_cameras(5, 2.5, 60.0, 13, 9)][1:3]
    inside = dict(cams[0])
    inside["R"], inside["t"] = np.eye(3), np.array([0.1, 0.05, 0.2])
    along = dict(inside)             # the middle pixel's ray runs along z alone
    along.update(t=np.array([0.0, 0.0, 2.0]), cx=6.5, cy=4.5)
    cams += [ocam.to_float32(inside), ocam.to_float32(along)]
    V = iso.Volume(torch.tensor(vol, device="cuda"))
    ctx = P.Context(0)
    imgs = iso.raycast(ctx, V, [P.camera_from_dict(c) for c in cams], level, step)
    again = iso.raycast(ctx, V, [P.camera_from_dict(c) for c in cams], level, step)
    torch.cuda.synchronize()
    with np.errstate(all="ignore"):
        want = [OI.raycast(vol, (-1, -1, -1), (1, 1, 1), level, c, step) for c in cams]
    for img, rep, w in zip(imgs, again, want):
        got = img.cpu().numpy().astype(np.float64)
        assert np.array_equal(np.isnan(got), np.isnan(w))
        assert np.nanmax(np.abs(got - w)) < 1e-5
        assert torch.equal(img.nan_to_num(), rep.nan_to_num())
    assert any(w.max() > 0 for w in want) or kind == "zero"


# ---------------------------------------------------------------- binning
@pytest.mark.parametrize("n", [
    1, 1023, 1025,                # one block of four keys a thread, and one key more
    65536, 65537,                 # digit tables summed by the scatter itself, then scanned
    524288, 524289,               # the gather's blocks leave the totals, then a launch does
    1048576, 1048577])            # four, then sixteen keys a thread
def test_binning_at_sort_sizes(P, ctx, n):
    """Records, ranges and counts of n Gaussians against a stable sort of the exported
    rectangles and depths (whole numbers: equal)."""
    g = torch.Generator("cuda").manual_seed(n)
    means = torch.rand((3, n), device="cuda", generator=g) * 3 - 1.5     # some off the view
    p = P.Params(means, torch.full((3, n), -4.6, device="cuda"),
                 torch.tensor([[1.], [0], [0], [0]], device="cuda").repeat(1, n).contiguous(),
                 torch.zeros(n, device="cuda"), torch.zeros((3, n), device="cuda"), 0)
    cam = P.orbit_cameras(4, 2.5, 60.0, 200, 120)[2]
    _, frame = P.render_fwd(ctx, p, [cam], tile=8, lds_depth=64)
    st = frame.stats()
    rect = frame.export("rects").view(n, 2).long() & 0xffffffff
    depth = frame.export("depths").long() & 0xffffffff
    x0, y0, x1, y1 = rect[:, 0] & 0xffff, rect[:, 0] >> 16, rect[:, 1] & 0xffff, rect[:, 1] >> 16
    w, h = (x1 - x0 + 1).clamp(min=0), (y1 - y0 + 1).clamp(min=0)
    m = w * h
    assert st["n_visible"] == int((m > 0).sum()) and st["n_records"] == int(m.sum())
    order = torch.sort(depth, stable=True)[1]
    e = torch.repeat_interleave(order, m[order])
    r = torch.arange(e.numel(), device="cuda") - torch.repeat_interleave(
        m[order].cumsum(0) - m[order], m[order])
    tile = (y0[e] + r // w[e].clamp(min=1)) * 25 + x0[e] + r % w[e].clamp(min=1)
    tile, by = torch.sort(tile, stable=True)
    assert torch.equal(frame.export("values").long(), e[by])
    assert torch.equal(frame.export("keys"), (tile << 32) | depth[e[by]])
    count = torch.bincount(tile, minlength=st["n_tiles"])
    end = count.cumsum(0)
    want = torch.stack([end - count, end], 1) * (count > 0)[:, None]
    assert torch.equal(frame.export("ranges").view(-1, 2).long(), want)
    frame.release()


@pytest.mark.parametrize("n,views", [(1, 1), (63, 1), (64, 1), (65, 2), (1025, 1), (4096, 3),
                                     (8192, 2), (16383, 1), (16385, 1)])
def test_binning_of_few_entries_with_equal_depths(P, ctx, n, views):
    """Depth order of few entries (placed by counting up to 16384 of them) where many depths
    are equal and some entries are off the view, against a stable sort (whole numbers:
    equal), and the records' total."""
    g = torch.Generator("cuda").manual_seed(n)
    means = torch.rand((3, n), device="cuda", generator=g) * 3 - 1.5
    means = (means * 4).round() / 4                    # few distinct places
    p = P.Params(means, torch.full((3, n), -3.6, device="cuda"),
                 torch.tensor([[1.], [0], [0], [0]], device="cuda").repeat(1, n).contiguous(),
                 torch.zeros(n, device="cuda"), torch.zeros((3, n), device="cuda"), 0)
    cams = P.orbit_cameras(4, 2.5, 60.0, 130, 70)[:views]
    _, frame = P.render_fwd(ctx, p, cams, tile=16, lds_depth=64)
    st = frame.stats()
    rect = frame.export("rects").view(-1, 2).long() & 0xffffffff
    depth = frame.export("depths").long() & 0xffffffff
    x0, y0, x1, y1 = rect[:, 0] & 0xffff, rect[:, 0] >> 16, rect[:, 1] & 0xffff, rect[:, 1] >> 16
    m = (x1 - x0 + 1).clamp(min=0) * (y1 - y0 + 1).clamp(min=0)
    assert depth.numel() == n * views
    assert st["n_visible"] == int((m > 0).sum()) and st["n_records"] == int(m.sum())
    order = torch.sort(depth, stable=True)[1]
    e = torch.repeat_interleave(order, m[order])
    r = torch.arange(e.numel(), device="cuda") - torch.repeat_interleave(
        m[order].cumsum(0) - m[order], m[order])
    wide = (x1 - x0 + 1).clamp(min=1)[e]
    tile = (e // n) * (9 * 5) + (y0[e] + r // wide) * 9 + x0[e] + r % wide
    tile, by = torch.sort(tile, stable=True)
    if e.numel():
        assert torch.equal(frame.export("values").long(), e[by])
        assert torch.equal(frame.export("keys"), (tile << 32) | depth[e[by]])
    frame.release()


@pytest.mark.parametrize("n,w,h,log_scale,fits", [
    (300_000, 2100, 2104, -5.6, True),     # 17-bit tile numbers
    (300_000, 4216, 4200, -6.6, True),     # 19-bit
    (2_000, 2100, 2104, -3.0, False),      # 17-bit, too many records for the wide digits' table
    (300_000, 1600, 1600, -5.6, None),     # 16-bit
])
def test_binning_of_many_tiles(P, ctx, n, w, h, log_scale, fits):
    """More than 2^20 records over more than 65536 tiles (sorted by wide digits where the
    entries' scratch holds their table) against a stable sort of the exported rectangles
    and depths (whole numbers: equal)."""
    g = torch.Generator("cuda").manual_seed(w)
    means = torch.rand((3, n), device="cuda", generator=g) * 2 - 1
    p = P.Params(means, torch.full((3, n), log_scale, device="cuda"),
                 torch.tensor([[1.], [0], [0], [0]], device="cuda").repeat(1, n).contiguous(),
                 torch.zeros(n, device="cuda"), torch.zeros((3, n), device="cuda"), 0)
    cam = P.orbit_cameras(4, 2.5, 60.0, w, h)[1]
    _, frame = P.render_fwd(ctx, p, [cam], tile=8, lds_depth=64)
    st = frame.stats()
    tiles, nx = st["n_tiles"], -(-w // 8)
    assert st["n_records"] > 1 << 20
    bits = (tiles - 1).bit_length()
    assert (bits > 16) == (fits is not None)
    if fits is not None:
        table = (1 << -(-bits // 2)) * (-(-st["n_records"] // 8192) + 4)
        assert (table <= n) if fits else (table > 2 * n)
    rect = frame.export("rects").view(n, 2).long() & 0xffffffff
    depth = frame.export("depths").long() & 0xffffffff
    x0, y0, x1, y1 = rect[:, 0] & 0xffff, rect[:, 0] >> 16, rect[:, 1] & 0xffff, rect[:, 1] >> 16
    m = (x1 - x0 + 1).clamp(min=0) * (y1 - y0 + 1).clamp(min=0)
    order = torch.sort(depth, stable=True)[1]
    e = torch.repeat_interleave(order, m[order])
    r = torch.arange(e.numel(), device="cuda") - torch.repeat_interleave(
        m[order].cumsum(0) - m[order], m[order])
    wide = (x1 - x0 + 1).clamp(min=1)[e]
    tile, by = torch.sort((y0[e] + r // wide) * nx + x0[e] + r % wide, stable=True)
    assert torch.equal(frame.export("values").long(), e[by])
    assert torch.equal(frame.export("keys"), (tile << 32) | depth[e[by]])
    frame.release()


# ---------------------------------------------------------------- outputs sized inside a call
def test_outputs_allocated_between_count_and_write(P, ctx, monkeypatch):
    """extract() and densify(), which allocate inside the library's call, against counting
    and then writing in two calls (equal); an allocation that fails ends the call."""
    import ctypes as C
    from paper_2509_05216_amd import _lib as L
    from paper_2509_05216_amd import density as D
    from paper_2509_05216_amd import iso
    null = None
    V = iso.Volume(torch.tensor(_volume("noise", (17, 12, 9)), device="cuda"))
    pts = iso.extract(ctx, V, 0.5, 0.6, 9)
    n = C.c_int64()
    two = torch.empty((3, iso.count(ctx, V, 0.5, 0.6, 9)), device="cuda")
    L.check(L.lib().gs_iso_extract(ctx.handle, V.abi(), 0.5, 0.6, 9, C.c_void_p(two.data_ptr()),
                                   two.shape[1], C.byref(n), null))
    assert n.value == pts.shape[1] and torch.equal(pts, two)
    assert iso.extract(ctx, V, 7.0).shape == (3, 0)
    assert L.lib().gs_iso_extract_alloc(ctx.handle, V.abi(), 0.5, 1.0, 0,
                                        L.PointsFn(lambda _, k: None), null, C.byref(n),
                                        null) == -2

    g = torch.Generator("cuda").manual_seed(3)
    r = lambda *s: torch.rand(s, device="cuda", generator=g)  # noqa: E731
    p, m, v = (P.Params(r(3, 700), r(3, 700) * 2 - 5, r(4, 700) - 0.5, r(700) * 6 - 4,
                        r(12, 700), 1) for _ in range(3))
    st = D.DensityStats(r(700) ** 3 * 2e-3, torch.ones(700, dtype=torch.int32, device="cuda"),
                        torch.zeros(700, dtype=torch.int32, device="cuda"))
    po, mo, vo, info, src = D.densify(ctx, p, m, v, st, 2.5, seed=5, want_src=True)
    k = info["n_out"]
    assert info["split"] > 0 and info["cloned"] > 0
    outs = [D._empty(k, 1, "cuda") for _ in range(3)]
    src2 = torch.empty(k, dtype=torch.int32, device="cuda")
    out = L.GsDensityInfo()
    L.check(L.lib().gs_densify(ctx.handle, p.abi(), m.abi(), v.abi(), st.abi(),
                               C.byref(D._opts(2.5, 5)), *(o.abi() for o in outs),
                               C.c_void_p(src2.data_ptr()), C.byref(out), null))
    assert D._info(out) == info and torch.equal(src, src2)
    for a, b in zip((po, mo, vo), outs):
        for x, y in zip(a.tensors(), b.tensors()):
            assert torch.equal(x, y)

    def full(*a, **kw):
        raise MemoryError("no room")
    monkeypatch.setattr(D, "_empty", full)
    with pytest.raises(MemoryError):
        D.densify(ctx, p, m, v, st, 2.5)


# ---------------------------------------------------------------- loss
@pytest.mark.parametrize("sizes", [
    [(32, 33)],                                  # one tile a block
    [(1003, 771)],                               # strips, ragged both ways
    [(33, 11000), (95, 31)],                     # long strips, two views in a launch
    [(700, 640), (5, 9), (640, 700)],            # views of one and of many strips together
    [(2200, 2000), (40, 50)]])                   # more than the shared workspace: one by one
def test_loss_strips_and_groups(P, ctx, sizes):
    """Loss, gradients and metrics against the float64 oracle (the tolerances of the
    small-image test)."""
    from oracle import loss as OL
    rng = np.random.default_rng(11)
    ys = [rng.random((3, h, w)).astype(np.float32) for w, h in sizes]
    xs = [np.clip(y + 0.2 * rng.standard_normal(y.shape), 0, 1).astype(np.float32) for y in ys]
    cams = [P.camera(np.eye(3), np.zeros(3), 200.0, 200.0, w / 2, h / 2, w, h) for w, h in sizes]
    gx, gy = ([torch.tensor(t, device="cuda") for t in ts] for ts in (xs, ys))
    loss, grads = P.loss_grad(ctx, gx, gy, cams)
    loss2, none = P.loss_grad(ctx, gx, gy, cams, want_grad=False)
    m = P.core.image_metrics(ctx, gx, gy, cams)
    torch.cuda.synchronize()
    assert none is None and torch.equal(loss, loss2)
    want, dl = OL.batch_loss([x.astype(np.float64) for x in xs],
                             [y.astype(np.float64) for y in ys], 0.2)
    assert abs(loss.item() - want) < 1e-5 * max(1, abs(want))
    for k, (x, y) in enumerate(zip(xs, ys)):
        assert rel_l2(grads[k].cpu().numpy(), dl[k]) < 1e-4
        l1 = np.abs(x.astype(np.float64) - y).mean()
        ssim = OL.ssim(x.astype(np.float64), y.astype(np.float64))
        assert abs(m[k, 2].item() - l1) < 1e-5 and abs(m[k, 3].item() - np.mean(ssim)) < 1e-5


# ---------------------------------------------------------------- tile order
@pytest.mark.parametrize("views,size,tile", [(9, (256, 240), 16), (3, (250, 179), 8),
                                             (16, (410, 310), 32)])
def test_tiles_in_length_order(P, ctx, views, size, tile):
    """Views rendered together, with at least 2048 tiles blended longest list first, against
    each view alone, blended in tile order: the same images and gradient sums."""
    import gsscenes
    p = P.Params.from_numpy(gsscenes.make_scene("iso1m", n=4000, G=96).params)
    cams = P.orbit_cameras(views, 2.5, 60.0, *size)
    assert views * -(-size[0] // tile) * -(-size[1] // tile) >= 2048
    assert -(-size[0] // tile) * -(-size[1] // tile) < 2048
    imgs, frame = P.render_fwd(ctx, p, cams, tile=tile, lds_depth=64)
    g = torch.Generator("cuda").manual_seed(1)
    dl = [torch.rand(i.shape, device="cuda", generator=g) for i in imgs]
    got = P.render_bwd(ctx, frame, p, dl)
    want = p.zeros_like()
    one = P.Frame()
    for k, c in enumerate(cams):
        img, _ = P.render_fwd(ctx, p, [c], tile=tile, lds_depth=64, frame=one)
        P.render_bwd(ctx, one, p, [dl[k]], want, accumulate=True)
        assert torch.equal(img[0], imgs[k]), k
    for a, b in zip(got.tensors(), want.tensors()):
        assert rel_l2(a.cpu().numpy(), b.cpu().numpy()) < 1e-5
    frame.release()


@pytest.mark.parametrize("n,degree", [(1, 0), (4096, 1), (5121, 2), (70_001, 3)])
def test_densify_with_and_without_room_for_classes(P, ctx, n, degree):
    """The writing pass reading the counting pass's classes, and (in a context whose scratch
    holds the offsets only) classifying again: equal; children and clones among them."""
    from paper_2509_05216_amd import density as D
    g = torch.Generator("cuda").manual_seed(n)
    r = lambda *s: torch.rand(s, device="cuda", generator=g)  # noqa: E731
    rows = 3 * (degree + 1) ** 2
    p, m, v = (P.Params(r(3, n), r(3, n) * 2 - 5, r(4, n) - 0.5, r(n) * 6 - 4, r(rows, n), degree)
               for _ in range(3))
    st = D.DensityStats(r(n) ** 3 * 2e-3, torch.ones(n, dtype=torch.int32, device="cuda"),
                        torch.zeros(n, dtype=torch.int32, device="cuda"))
    small = P.Context(0, mem_budget=4096)
    a = D.densify(ctx, p, m, v, st, 2.5, seed=5, want_src=True)
    b = D.densify(small, p, m, v, st, 2.5, seed=5, want_src=True)
    assert a[3] == b[3] and (n < 1000 or (a[3]["cloned"] and a[3]["split"]))
    assert torch.equal(a[4], b[4])
    for x, y in zip(a[:3], b[:3]):
        for t, u in zip(x.tensors(), y.tensors()):
            assert torch.equal(t, u)
    small.close()


# ---------------------------------------------------------------- ray-cast at the limits of float32
def _cast_and_check(P, vol, level, step, cams, lo=(-1.0, -1.0, -1.0), hi=(1.0, 1.0, 1.0)):
    """One ray-cast against the float64 oracle's images, which it returns."""
    from oracle import iso as OI
    from paper_2509_05216_amd import iso
    step, level = float(np.float32(step)), float(np.float32(level))
    V = iso.Volume(torch.tensor(vol, device="cuda"), lo, hi)
    imgs = iso.raycast(P.Context(0), V, [P.camera_from_dict(c) for c in cams], level, step)
    torch.cuda.synchronize()
    with np.errstate(all="ignore"):
        want = [OI.raycast(vol, lo, hi, level, c, step) for c in cams]
    for img, w in zip(imgs, want):
        got = img.cpu().numpy().astype(np.float64)
        assert np.array_equal(np.isnan(got), np.isnan(w))
        assert np.nanmax(np.abs(got - w)) < 1e-5
    return want


@pytest.mark.parametrize("shape,step", [((7, 6, 400), 0.005), ((9, 8, 7), 0.05)])
@pytest.mark.parametrize("size,level", [
    (3.2e38, 0.5),                  # differences of corners pass the largest float32
    (2e38, -1e38), (5e36, 3e38),
    (1e-42, 0.0), (3e-44, 0.0),     # subnormal: float32 rounds by a fixed amount
    (1e-42, 2e-43), (1e-36, 0.0)])
def test_raycast_of_very_large_and_subnormal_values(P, shape, step, size, level):
    """Rays through volumes whose values leave the range in which a float32 sample's error
    follows the size of the values, through cell classes (the long volume) and without."""
    from oracle import camera as ocam
    rng = np.random.default_rng(11)
    vol = (rng.uniform(-1, 1, shape) * size).astype(np.float32)
    assert np.isfinite(vol).all()
    cams = [ocam.to_float32(c) for c in ocam.orbit_cameras(5, 2.5, 60.0, 13, 9)][1:3]
    want = _cast_and_check(P, vol, level, step, cams)
    assert any(w.max() > 0 for w in want) or abs(level) > size


@pytest.mark.parametrize("nz", [9, 400])
@pytest.mark.parametrize("nx,nan_from,nan_to", [
    (59, 30, 59),      # sample in cell 29; its coordinate by reciprocal falls into cell 28
    (51, 0, 25)])      # sample in cell 24; by reciprocal in cell 25
def test_raycast_beside_values_that_are_not_finite(P, nx, nan_from, nan_to, nz):
    """A ray along a grid plane whose cells are finite on one side only: the cell of a sample
    is that of the float64 division, whose NaN hides the surface."""
    lo, hi, x0 = (-0.75, -1.0, -1.0), (1.0, 1.0, 1.0), 0.125
    h = (hi[0] - lo[0]) / (nx - 1)
    assert np.floor((x0 - lo[0]) / h) != np.floor((x0 - lo[0]) * (1.0 / h))
    z = np.linspace(0, 1, nz, dtype=np.float32)[:, None, None]
    vol = np.broadcast_to(z, (nz, 5, nx)).copy()
    cam = dict(R=np.eye(3), t=np.array([-x0, 0.1, 2.0]), fx=10.0, fy=10.0, cx=0.5, cy=0.5,
               width=1, height=1, z_near=0.2)
    step = 0.05 if nz == 9 else 0.005
    assert _cast_and_check(P, vol, 0.43, step, [cam], lo, hi)[0].max() > 0   # finite: a surface
    vol[:, :, nan_from:nan_to] = np.nan
    assert _cast_and_check(P, vol, 0.43, step, [cam], lo, hi)[0].max() == 0


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("kind", ["rendered", "target", "gradient"])
def test_loss_of_views_whose_buffers_overlap(P, ctx, kind, noalloc):
    """A view's gradient written over part of the next view's image, target or gradient: the
    views are taken one after the other, so the next one reads (or writes) it as it is then."""
    h, w = 61, 93
    n, off = 3 * h * w, 1000
    g = torch.Generator("cuda").manual_seed(5)
    x0, x1, y0, y1 = (torch.rand((3, h, w), device="cuda", generator=g) for _ in range(4))
    cams = [P.camera(np.eye(3), np.zeros(3), 200.0, 200.0, w / 2, h / 2, w, h)] * 2

    def call(xs, ys, dl):
        loss = torch.zeros(1, device="cuda")
        P.loss_grad_into(ctx, xs, ys, cams, loss, dl, 0.2, noalloc=noalloc)
        torch.cuda.synchronize()
        return loss

    buf = torch.zeros(n + off, device="cuda")
    over, first = buf[:n].view(3, h, w), buf[off:].view(3, h, w)
    d0, d1, e1 = (torch.zeros((3, h, w), device="cuda") for _ in range(3))
    call([x0, x1], [y0, y1], [d0, d1])             # the first view's gradient, apart
    if kind == "gradient":
        call([x0, x1], [y0, y1], [first, over])
        assert torch.equal(over, d1)               # the second view's is written last
        assert torch.equal(buf[n:], d0.view(-1)[n - off:])
        return
    hit = (x1 if kind == "rendered" else y1).clone()
    over.copy_(hit)
    hit.view(-1)[off:] = d0.view(-1)[:n - off]     # what the second view finds
    want = call([x0, hit if kind == "rendered" else x1], [y0, y1 if kind == "rendered" else hit],
                [d0, e1])
    got = call([x0, over if kind == "rendered" else x1],
               [y0, y1 if kind == "rendered" else over], [first, d1])
    assert torch.equal(first, d0) and torch.equal(d1, e1) and torch.equal(got, want)
