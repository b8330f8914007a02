"""Scratch that only makes a call faster: it gives way to memory that a call cannot do
without, and asking for it in vain changes nothing."""
import numpy as np
import pytest
import torch

import gsscenes

pytestmark = pytest.mark.gpu

SLACK = 256 << 10


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2509_05216_amd as P
    return P


@pytest.fixture(scope="module")
def scene(P):
    p = P.Params.from_numpy(gsscenes.make_scene("iso1m", n=60_000, G=96).params)
    cams = P.orbit_cameras(2, 2.5, 60.0, 160, 120)
    c = P.Context(0)
    imgs, frame = P.render_fwd(c, p, cams)
    torch.cuda.synchronize()
    return p, cams, imgs, c.memory()[0]


def _loss_views(P, sizes):
    g = torch.Generator("cuda").manual_seed(2)
    xs, ys = ([torch.rand((3, h, w), device="cuda", generator=g) for w, h in sizes]
              for _ in range(2))
    return xs, ys, [P.camera(np.eye(3), np.zeros(3), 200.0, 200.0, w / 2, h / 2, w, h)
                    for w, h in sizes]


def _call(P, kind):
    """(call of a context that returns tensors, bytes of scratch it cannot do without)."""
    from paper_2509_05216_amd import density as D
    from paper_2509_05216_amd import iso
    c = P.Context(0)
    if kind == "loss":
        xs, ys, cams = _loss_views(P, [(400, 300)] * 3)
        P.loss_grad(c, xs[:1], ys[:1], cams[:1])
        return (lambda ctx: [P.loss_grad(ctx, xs, ys, cams)[0], *P.loss_grad(ctx, xs, ys, cams)[1]],
                c.memory()[0])
    if kind == "raycast":
        a = torch.linspace(-1, 1, 256, device="cuda")
        vol = (1.2 - (a[:, None, None] ** 2 + a[:, None] ** 2 + a ** 2).sqrt()).contiguous()
        V, cams = iso.Volume(vol), P.orbit_cameras(2, 2.5, 60.0, 64, 48)
        return lambda ctx: iso.raycast(ctx, V, cams, 0.5, 0.008), 0
    n = 1_000_000
    g = torch.Generator("cuda").manual_seed(3)
    r = lambda *s: torch.rand(s, device="cuda", generator=g)  # noqa: E731
    p, m, v = (P.Params(r(3, n), r(3, n) * 2 - 5, r(4, n) - 0.5, r(n) * 6 - 4, r(3, n), 0)
               for _ in range(3))
    st = D.DensityStats(r(n) ** 3 * 2e-3, torch.ones(n, dtype=torch.int32, device="cuda"),
                        torch.zeros(n, dtype=torch.int32, device="cuda"))
    return (lambda ctx: [t for q in D.densify(ctx, p, m, v, st, 2.5, seed=5)[:3]
                         for t in q.tensors()], 64 << 10)


@pytest.mark.parametrize("kind", ["loss", "raycast", "densify"])
def test_optional_scratch_gives_way_to_a_forward(P, scene, kind):
    """A context whose budget holds a frame and the least scratch of another call together:
    that call, which takes more while there is room, then the forward, then both again."""
    p, cams, ref, frame_bytes = scene
    call, least = _call(P, kind)
    want = [t.clone() for t in call(P.Context(0))]
    ctx = P.Context(0, mem_budget=frame_bytes + least + SLACK)
    first = call(ctx)
    assert ctx.memory()[0] > least + SLACK          # the optional part was taken
    imgs, frame = P.render_fwd(ctx, p, cams)
    again = call(ctx)
    imgs2, frame = P.render_fwd(ctx, p, cams, frame=frame)
    torch.cuda.synchronize()
    assert ctx.memory()[0] <= frame_bytes + least + SLACK
    for a, b, c in zip(first, again, want):
        assert torch.equal(a, c) and torch.equal(b, c)
    for a, b, c in zip(imgs, imgs2, ref):
        assert torch.equal(a, c) and torch.equal(b, c)


@pytest.mark.parametrize("kind", ["loss", "raycast", "densify"])
def test_a_refused_optional_size_changes_nothing(P, scene, kind):
    """A call without room for its optional scratch leaves kept frames and the thread's last
    error as they are."""
    from paper_2509_05216_amd import _lib as L
    p, cams, _, frame_bytes = scene
    call, least = _call(P, kind)
    want = [t.clone() for t in call(P.Context(0))]
    ctx = P.Context(0, mem_budget=frame_bytes + least + SLACK)
    P.render_fwd(ctx, p, cams)[1].release()         # kept
    held = ctx.memory()[0]
    assert L.lib().gs_orbit_cameras(0, 2.5, 60.0, 64, 64, (L.GsCamera * 1)()) == -1
    text = L.lib().gs_last_error()
    for _ in range(2):
        got = call(ctx)
        assert ctx.memory()[0] >= held
        assert L.lib().gs_last_error() == text
    for a, b in zip(got, want):
        assert torch.equal(a, b)


def test_captured_loss_takes_the_workspace_as_it_is(P):
    """An eager loss call recorded into a caller's graph: the workspace holds one view at a
    time, so nothing is allocated, though all views together would like more."""
    ctx = P.Context(0)
    for sizes in ([(1, 16384)], [(500, 400)]):      # rows of tiles, pixels
        xs, ys, cams = _loss_views(P, sizes)
        P.loss_grad(ctx, xs, ys, cams)
    xs, ys, cams = _loss_views(P, [(400, 300)] * 3)
    want, dl = P.loss_grad(P.Context(0), xs, ys, cams)
    loss, got = torch.zeros(1, device="cuda"), [torch.zeros_like(x) for x in xs]
    torch.cuda.synchronize()
    held = ctx.memory()[0]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        P.loss_grad_into(ctx, xs, ys, cams, loss, got, 0.2)
    assert ctx.memory()[0] == held
    for rep in range(3):
        loss.zero_()
        for t in got:
            t.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(loss.view(-1), want.view(-1)), rep
        for a, b in zip(got, dl):
            assert torch.equal(a, b), rep


@pytest.mark.parametrize("n,side,tile,log_scale,less", [
    (3_000, 1024, 8, -4.5, 60 << 10),       # the tile order, of more tiles than entries
    (20_000, 1024, 8, -3.9, 500 << 10),     # digit tables of four keys a thread
    (20_000, 400, 16, -4.5, 0)])
def test_forward_without_room_for_faster_sorts(P, n, side, tile, log_scale, less):
    """A budget short of what a frame takes without one by memory that only makes its sorts
    and its schedule faster: the same frame, images and gradients."""
    g = torch.Generator("cuda").manual_seed(n + side)
    r = lambda *s: torch.rand(s, device="cuda", generator=g)  # noqa: E731
    ls = log_scale + torch.tensor([[0.2], [0.0], [-0.2]], device="cuda").repeat(1, n)
    p = P.Params(r(3, n) * 1.6 - 0.8, ls.contiguous(), r(4, n) - 0.5, r(n) * 4 - 2, r(3, n), 0)
    cams = P.orbit_cameras(3, 2.5, 60.0, side, side)[1:2]
    free = P.Context(0)
    want, frame = P.render_fwd(free, p, cams, tile=tile, lds_depth=64)
    torch.cuda.synchronize()
    total, st = free.memory()[0], frame.stats()
    assert (st["n_records"] > 1 << 19) == (n > 3000 and side > 400)
    tight = P.Context(0, mem_budget=total - less)
    imgs, frame2 = P.render_fwd(tight, p, cams, tile=tile, lds_depth=64)
    assert torch.equal(imgs[0], want[0])
    st2 = frame2.stats()
    assert all(st[k] == st2[k] for k in st if k != "device_bytes")
    for k in ("keys", "values", "ranges"):
        assert torch.equal(frame.export(k), frame2.export(k)), k
    dl = [r(3, side, side)]
    a, b = P.render_bwd(free, frame, p, dl), P.render_bwd(tight, frame2, p, dl)
    torch.cuda.synchronize()
    for x, y in zip(a.tensors(), b.tensors()):
        assert (x - y).abs().max().item() <= 1e-5 * max(y.abs().max().item(), 1e-6)
