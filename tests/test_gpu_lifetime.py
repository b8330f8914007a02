"""Object lifetimes across the C ABI: a context destroyed while a frame it
created is alive stays usable by that frame, and is freed by the frame's
release; a later context on the device works normally."""
import ctypes as C

import numpy as np
import pytest
import torch

import gsscenes
from oracle import camera as ocam

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2509_05216_amd as P
    return P


def _render_raw(P, ctx_handle, params, cam, img, frame_handle):
    from paper_2509_05216_amd import _lib as L
    from paper_2509_05216_amd.core import _cam_array, _opts
    pa, keep = L.ptr_array([img.data_ptr()])
    o = _opts(16, 256, (0.0, 0.0, 0.0), 0)
    return L.lib().gs_render_fwd(ctx_handle, params.abi(), _cam_array([cam]), 1, pa, C.byref(o),
                                 C.byref(frame_handle), None)


def test_frame_outlives_destroyed_context(P):
    from paper_2509_05216_amd import _lib as L
    lib = L.lib()
    scene = gsscenes.make_scene("tiny", n=2000)
    params = P.Params.from_numpy(scene.params)
    cam = P.camera_from_dict(ocam.to_float32(ocam.orbit_cameras(4, 2.5, 60.0, 96, 80)[1]))
    ref, _ = P.render_fwd(P.Context(0), params, [cam])
    torch.cuda.synchronize()

    h = C.c_void_p()
    assert lib.gs_ctx_create(0, C.c_size_t(0), C.byref(h)) == 0
    img = torch.empty((3, 80, 96), device="cuda")
    fr = C.c_void_p()
    assert _render_raw(P, h, params, cam, img, fr) == 0
    torch.cuda.synchronize()
    lib.gs_ctx_destroy(h)                      # the frame still holds the context
    st = L.GsFrameStats()
    assert lib.gs_frame_stats_get(fr, C.byref(st)) == 0
    assert st.n_gaussians == 2000 and st.n_records > 0
    out = torch.empty(st.n_pixels, dtype=torch.int32, device="cuda")
    assert lib.gs_frame_export(fr, L.EXPORT["n_contrib"], -1, C.c_void_p(out.data_ptr()),
                               C.c_size_t(out.numel() * 4), None) == 0
    torch.cuda.synchronize()
    lib.gs_frame_release(fr)                   # frees the context too
    assert torch.equal(img, ref[0])

    # a new context on the same device is unaffected
    imgs, frame = P.render_fwd(P.Context(0), params, [cam])
    torch.cuda.synchronize()
    assert torch.equal(imgs[0], ref[0])
    frame.release()


def _views(P, sizes, start=0):
    return [P.camera_from_dict(ocam.to_float32(ocam.orbit_cameras(8, 2.5, 60.0, W, H)[start + i]))
            for i, (W, H) in enumerate(sizes)]


def test_graph_keeps_its_loss_workspace(P):
    """A captured step owns its loss workspace: a second graph on larger views and
    eager loss calls on a larger image (which grow the context's own workspace)
    must not disturb the replays of the first graph, which stay equal to the
    eager step on its views."""
    ctx = P.Context(0)
    scene = gsscenes.make_scene("tiny", n=3000)
    params = P.Params.from_numpy(scene.params)
    rng = np.random.default_rng(12)
    small = _views(P, [(96, 80), (64, 64)])
    tgt = [torch.tensor(rng.random((3, c.height, c.width)), dtype=torch.float32, device="cuda")
           for c in small]
    ga = P.StepGraph(ctx, params, small, tgt, with_adam=False)
    big = _views(P, [(320, 288), (256, 256)], start=2)
    tgt_b = [torch.tensor(rng.random((3, c.height, c.width)), dtype=torch.float32,
                          device="cuda") for c in big]
    gb = P.StepGraph(ctx, params, big, tgt_b, with_adam=False)
    # eager reference of graph A's step
    grads = params.zeros_like()
    imgs, frame = P.render_fwd(ctx, params, small)
    loss, dl = P.loss_grad(ctx, imgs, tgt, small)
    P.render_bwd(ctx, frame, params, dl, grads)
    torch.cuda.synchronize()
    ref_dl = [d.clone() for d in dl]
    huge = _views(P, [(640, 600)], start=5)
    x = torch.rand((3, 600, 640), device="cuda")
    for rep in range(3):
        gb.run()
        # an eager loss on a larger image than any graph's: the context workspace grows
        P.loss_grad(ctx, [x], [x * 0.5], huge)
        ga.run()
        torch.cuda.synchronize()
        for a, b in zip(ga.images, imgs):
            assert torch.equal(a, b), rep
        assert ga.loss.item() == loss.item(), rep
        for a, b in zip(ga.dl, ref_dl):
            assert torch.equal(a, b), rep
        for a, b in zip(ga.grads.tensors(), grads.tensors()):
            d = (a - b).abs().max().item()
            assert d <= 1e-5 * max(b.abs().max().item(), 1e-6), rep
    ga.close()
    gb.close()
    frame.release()


def test_server_first_batches_on_fresh_slots(P):
    """Each slot's first batch runs on a fresh frame (its device words cleared on
    the slot's own stream): a burst of requests that reaches every slot at once
    gives the images of eager rendering."""
    ctx = P.Context(0)
    a = gsscenes.make_scene("tiny", n=4000)
    b = gsscenes.make_scene("iso1m", n=3000, G=96)
    params = [P.Params.from_numpy(a.params), P.Params.from_numpy(b.params)]
    sizes = [(128, 96), (96, 96), (160, 128), (80, 64), (112, 112), (64, 48)]
    reqs = [(i % 2, c) for i, c in enumerate(_views(P, sizes))]
    refs = []
    for sid, cam in reqs:
        imgs, fr = P.render_fwd(ctx, params[sid], [cam])
        refs.append(imgs[0])
        fr.release()
    torch.cuda.synchronize()
    for trial in range(2):
        srv = P.Server(ctx, n_slots=6, max_batch_views=1)
        ids = [srv.add_scene(p) for p in params]
        tickets = [srv.submit(ids[sid], cam) for sid, cam in reqs]
        srv.drain()
        torch.cuda.synchronize()
        for (t, out), ref in zip(tickets, refs):
            assert torch.equal(out, ref), trial
        srv.close()


def test_entry_limit_is_checked_before_any_launch(P):
    """views x Gaussians past the frame's entry limit (2^32 - 2^20) is rejected with
    GS_ERR_CAPACITY on the host, before the parameters are touched (the count is set
    in the ABI struct; the arrays hold one Gaussian)."""
    from paper_2509_05216_amd import _lib as L
    from paper_2509_05216_amd.core import _cam_array, _opts
    ctx = P.Context(0)
    small = P.Params.from_numpy(gsscenes.make_scene("tiny", n=1000).params)
    ab = small.abi()
    ab.n = 1 << 28                           # 16 views x 2^28 = 2^32 > the limit
    cams = [P.camera_from_dict(c) for c in
            [ocam.to_float32(x) for x in ocam.orbit_cameras(16, 2.5, 60.0, 64, 64)]]
    imgs = [torch.empty((3, 64, 64), device="cuda") for _ in cams]
    pa, keep = L.ptr_array([t.data_ptr() for t in imgs])
    o = _opts(16, 256, (0.0, 0.0, 0.0), 0)
    fr = C.c_void_p()
    st = L.lib().gs_render_fwd(ctx.handle, ab, _cam_array(cams), 16, pa, C.byref(o),
                               C.byref(fr), None)
    assert st == -4, L.lib().gs_last_error()
    assert b"exceeds" in L.lib().gs_last_error()
    assert not fr.value
    ctx.close()


def _step(P, ctx, params, cams, dl, frame=None, **kw):
    _, frame = P.render_fwd(ctx, params, cams, frame=frame)
    return P.render_bwd(ctx, frame, params, dl, **kw), frame


def test_kept_sums_do_not_reach_a_later_larger_forward(P):
    """Screen-space sums kept in a frame are cleared by the next forward only as far as
    that one reaches; a later, larger forward on the frame still starts from zeros."""
    ctx = P.Context(0)
    big = P.Params.from_numpy(gsscenes.make_scene("tiny", n=3000).params)
    small = P.Params.from_numpy(gsscenes.make_scene("tiny", n=700).params)
    cams = _views(P, [(96, 80), (96, 80)])
    dl = [torch.rand((3, 80, 96), device="cuda", generator=torch.Generator("cuda").manual_seed(i))
          for i in range(2)]
    ref, fresh = _step(P, ctx, big, cams, dl)
    _, frame = _step(P, ctx, big, cams, dl, keep_screen=True)
    _step(P, ctx, small, cams, dl, frame)
    got, _ = _step(P, ctx, big, cams, dl, frame)
    torch.cuda.synchronize()
    for a, b in zip(got.tensors(), ref.tensors()):
        assert (a - b).abs().max().item() <= 1e-5 * max(b.abs().max().item(), 1e-6)
    frame.release()
    fresh.release()
    ctx.close()


def test_released_frames_are_reused_and_given_back(P):
    """A released frame's buffers serve the next new frame of the context (of another
    shape, on another stream) with the results of a fresh context, are given up when the
    context's budget needs them, and hold no more than four frames."""
    big = P.Params.from_numpy(gsscenes.make_scene("tiny", n=6000).params)
    small = P.Params.from_numpy(gsscenes.make_scene("tiny", n=900).params)
    shapes = [(big, _views(P, [(160, 96)] * 3)), (small, _views(P, [(64, 48)])),
              (big, _views(P, [(80, 112)] * 2, start=3))]
    refs = []
    for p, cams in shapes:
        c = P.Context(0)
        dl = [torch.full((3, k.height, k.width), 0.3, device="cuda") for k in cams]
        g, f = _step(P, c, p, cams, dl)
        torch.cuda.synchronize()
        refs.append((P.render_fwd(c, p, cams, frame=f)[0], g, dl))
    ctx = P.Context(0)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    for trial in range(2):
        for (p, cams), (imgs, g, dl) in zip(shapes, refs):
            stream = side if trial else torch.cuda.current_stream()
            with torch.cuda.stream(stream):
                got, frame = P.render_fwd(ctx, p, cams)
                gg = P.render_bwd(ctx, frame, p, dl)
                stream.synchronize()
            for a, b in zip(got, imgs):
                assert torch.equal(a, b)
            for a, b in zip(gg.tensors(), g.tensors()):
                assert (a - b).abs().max().item() <= 1e-5 * max(b.abs().max().item(), 1e-6)
            held = ctx.memory()[0]
            frame.release()
            assert ctx.memory()[0] == held          # kept for the next frame
    frames = [P.render_fwd(ctx, small, shapes[1][1])[1] for _ in range(6)]
    before = ctx.memory()[0]
    for f in frames:
        f.release()
    assert ctx.memory()[0] < before                 # two of the six were freed
    ctx.close()
    # a budget that holds one large frame and not a second beside it
    c0 = P.Context(0)
    _, f = P.render_fwd(c0, big, shapes[0][1])
    one = c0.memory()[0]
    f.release()
    c1 = P.Context(0, mem_budget=int(1.3 * one))
    _, f = P.render_fwd(c1, small, shapes[1][1])
    f.release()
    _, f2 = P.render_fwd(c1, big, shapes[2][1])
    f2.release()
    imgs, f3 = P.render_fwd(c1, big, shapes[0][1])  # larger than f2: the pool gives way
    torch.cuda.synchronize()
    for a, b in zip(imgs, refs[0][0]):
        assert torch.equal(a, b)
    assert c1.memory()[0] <= int(1.3 * one)
    f3.release()


def test_release_waits_for_every_stream_of_the_frame(P):
    """A frame used on two streams, the first still at work when it is released: the next
    forward, which takes over its buffers, does not reach the first stream's results."""
    ctx = P.Context(0)
    one = P.Params.from_numpy(gsscenes.make_scene("tiny", n=6000).params)
    two = P.Params.from_numpy(gsscenes.make_scene("iso1m", n=6000, G=96).params)
    cams = _views(P, [(160, 96)] * 3)
    _, frame = P.render_fwd(ctx, one, cams)
    want = [frame.export(k) for k in ("splats", "rects")]
    side, other = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        torch.cuda._sleep(300_000_000)
        got = [frame.export(k) for k in ("splats", "rects")]
    with torch.cuda.stream(other):
        frame.export("depths")
    held = ctx.memory()[0]
    frame.release()
    _, again = P.render_fwd(ctx, two, cams)
    torch.cuda.synchronize()
    assert ctx.memory()[0] <= 1.2 * held        # the released frame's buffers, not new ones
    for a, b in zip(got, want):
        assert torch.equal(a, b)
    again.release()
    ctx.close()


def test_a_small_forward_leaves_a_large_kept_frame(P):
    """A released frame much larger than a new forward needs stays for a forward of its own
    size; trim() gives back what is kept."""
    n = 500_000
    g = torch.Generator("cuda").manual_seed(1)
    r = lambda *s: torch.rand(s, device="cuda", generator=g)  # noqa: E731
    big = P.Params(r(3, n) - 0.5, r(3, n) - 6, r(4, n) - 0.5, r(n), r(3, n), 0)
    small = P.Params.from_numpy(gsscenes.make_scene("tiny", n=900).params)
    cams = _views(P, [(160, 96)] * 2)
    ctx = P.Context(0)
    want, frame = P.render_fwd(ctx, big, cams)
    large = frame.stats()["device_bytes"]
    assert large > 64 << 20
    frame.release()
    _, little = P.render_fwd(ctx, small, cams)
    assert little.stats()["device_bytes"] < 64 << 20
    before = ctx.memory()[0]
    again, frame = P.render_fwd(ctx, big, cams)
    assert ctx.memory()[0] == before and frame.stats()["device_bytes"] == large
    torch.cuda.synchronize()
    for a, b in zip(again, want):
        assert torch.equal(a, b)
    frame.release()
    ctx.trim()
    assert ctx.memory()[0] == little.stats()["device_bytes"]
    dl = [torch.ones((3, 96, 160), device="cuda")] * 2     # a frame in use is untouched
    ref, fresh = _step(P, P.Context(0), small, cams, dl)
    for a, b in zip(P.render_bwd(ctx, little, small, dl).tensors(), ref.tensors()):
        assert (a - b).abs().max().item() <= 1e-5 * max(b.abs().max().item(), 1e-6)
    little.release()
    fresh.release()
    ctx.trim()
    assert ctx.memory()[0] == 0
    ctx.close()
