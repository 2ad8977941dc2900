"""Calls between and inside other calls: plain renders beside a captured step,
and calls on a stream that the caller is capturing."""
import contextlib
import gc

import pytest

from paper_2406_02518_amd import binding, synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _view(az=0.0, w=40, h=33):
    return synth.view(w, h, 0.9, 1000.0, 600.0, az)


def _renderer():
    return binding.Renderer(0, stream=torch.cuda.Stream())


def _scene(n, seed=31):
    return synth.random_scene(seed, n, k=4, L=1, extent=18.0)


@contextlib.contextmanager
def _capturing(stream):
    """A graph that the caller captures on the stream.  No garbage is collected
    meanwhile: a graph destroyed then (torch synchronises the device for it) would
    end the process."""
    gc.collect()
    gc.disable()
    graph = torch.cuda.CUDAGraph()
    try:
        with torch.cuda.stream(stream):
            graph.capture_begin(capture_error_mode="thread_local")
            try:
                yield graph
            finally:
                graph.capture_end()
    finally:
        gc.enable()


def _status(call):
    """The status of the error that the call raises (no reference to it is kept)."""
    try:
        call()
    except binding.DDGSError as e:
        return e.status
    return binding.OK


def _capture(r, capacity):
    r.set_options(capacity=capacity)
    P = r.image_size()
    s = {"img": torch.empty(P, device="cuda"), "dl": torch.empty(P, device="cuda"),
         "loss": torch.empty(len(r.views), device="cuda"), "grads": r.alloc_grads(),
         "w": torch.sin(torch.arange(P, device="cuda", dtype=torch.float32))}
    torch.cuda.synchronize()
    with torch.cuda.stream(r.stream):
        binding.ddgs_step_capture(r.ctx, binding.LOSS_LINEAR, s["w"].data_ptr(), 0.0, s["img"].data_ptr(),
                                  s["dl"].data_ptr(), s["loss"].data_ptr(), r.grads_struct(s["grads"]))
    return s


def _fresh(sc, views, w):
    """Image, gradients and entry total from a renderer of their own."""
    r = _renderer()
    try:
        r.set_scene(sc)
        r.set_views(views)
        img = r.render().clone()
        g = {k: v.clone() for k, v in r.backward(w).items()}
        torch.cuda.synchronize()
        return img, g, r.num_rendered()
    finally:
        r.close()


@pytest.mark.parametrize("n,w,h", [(2000, 64, 64), (700, 40, 33), (9000, 60, 52)])
def test_plain_render_between_replays(n, w, h):
    """A step captured with an explicit capacity that fits (there is no sizing
    render), a plain render of the same scene, whose one-workgroup binning would
    take every tile of every Gaussian, and the replays behind it: the same
    results, with what the renderer may have freed in other tensors' hands."""
    sc, views = _scene(n), [_view(10.0, w, h)]
    wt = torch.sin(torch.arange(w * h, device="cuda", dtype=torch.float32))
    exp, exp_g, need = _fresh(sc, views, wt)
    r = _renderer()
    try:
        r.set_scene(sc)
        r.set_views(views)
        s = _capture(r, need + 100)
        for _ in range(3):
            assert torch.equal(r.render(), exp)
            torch.cuda.synchronize()
            others = [torch.full((sz,), 7.0, device="cuda") for sz in (1 << 12, 1 << 16, 1 << 18, 1 << 20)]
            s["img"].zero_()
            for g in s["grads"].values():
                g.zero_()
            torch.cuda.synchronize()
            binding.ddgs_step_launch(r.ctx)
            assert r.check_step() == 0
            torch.cuda.synchronize()
            assert torch.equal(s["img"], exp)
            for k in exp_g:
                assert torch.equal(s["grads"][k], exp_g[k]), k
            assert all(bool((x == 7.0).all()) for x in others)
    finally:
        r.close()


@pytest.mark.parametrize("n", [2000, 9000])
def test_plain_render_that_outgrows_a_step_drops_it(n):
    """A plain render that needs more entries than the step was captured for moves
    the buffers that the step holds: the launch is refused, and a new capture
    works."""
    sc, views = _scene(n), [_view(10.0, 60, 52)]
    exp, _, need = _fresh(sc, views, torch.ones(60 * 52, device="cuda"))
    r = _renderer()
    try:
        r.set_scene(sc)
        r.set_views(views)
        _capture(r, need // 4)
        assert torch.equal(r.render(), exp)
        assert _status(lambda: binding.ddgs_step_launch(r.ctx)) == binding.ERR_STATE
        s = _capture(r, need)
        binding.ddgs_step_launch(r.ctx)
        assert r.check_step() == 0
        torch.cuda.synchronize()
        assert torch.equal(s["img"], exp)
    finally:
        r.close()


def _refused(r, calls):
    """Runs the calls on r's stream while it is being captured; each is refused, and
    the graph around them stays whole."""
    spare = torch.zeros(8, device="cuda")
    torch.cuda.synchronize()
    with _capturing(r.stream) as graph:
        spare.add_(1.0)
        got = [_status(call) for call in calls]
    assert got == [binding.ERR_HIP] * len(calls)
    for _ in range(3):
        graph.replay()
    torch.cuda.synchronize()
    assert torch.equal(spare, torch.full_like(spare, 3.0))


@pytest.mark.parametrize("n", [500, 12000])
@pytest.mark.parametrize("fresh", [False, True])
def test_refused_calls_leave_the_views_to_the_next_render(n, fresh):
    """New views set before a call that a capturing stream refuses: nothing of the
    call goes into the graph, and the render behind the capture sees these views."""
    sc, old, new = _scene(n), [_view(10.0)], [_view(55.0)]
    exp, _, _ = _fresh(sc, new, torch.ones(40 * 33, device="cuda"))
    other, _, _ = _fresh(sc, old, torch.ones(40 * 33, device="cuda"))
    assert not torch.equal(exp, other)
    r = _renderer()
    try:
        r.set_scene(sc)
        if not fresh:
            r.set_views(old)
            r.render()
        r.set_views(new)
        P = r.image_size()
        out = [torch.empty(P, device="cuda") for _ in range(3)]
        loss, grads = torch.empty(1, device="cuda"), r.alloc_grads()
        calls = [lambda: binding.ddgs_render(r.ctx, out[0].data_ptr()),
                 lambda: binding.ddgs_step_capture(r.ctx, binding.LOSS_LINEAR, out[0].data_ptr(), 0.0,
                                                   out[1].data_ptr(), out[2].data_ptr(), loss.data_ptr(),
                                                   r.grads_struct(grads)),
                 lambda: binding.ddgs_autotune(r.ctx)]
        for c in calls:
            _refused(r, [c])
        _refused(r, calls)
        assert torch.equal(r.render(), exp)
    finally:
        r.close()


def test_empty_model_renders_into_a_graph():
    """Nothing is read back for an empty model: its render goes into the caller's
    graph, unless there are views to upload first."""
    r = _renderer()
    try:
        sc = synth.random_scene(3, 0, k=4, L=1)
        r.set_scene(sc)
        r.set_views([_view()])
        out = r.render()
        assert not out.any()
        torch.cuda.synchronize()
        with _capturing(r.stream) as graph:
            binding.ddgs_render(r.ctx, out.data_ptr())
        for _ in range(3):
            out.fill_(5.0)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert not out.any()
        r.set_views([_view(30.0)])
        _refused(r, [lambda: binding.ddgs_render(r.ctx, out.data_ptr())])
        assert not r.render().any()
    finally:
        r.close()


@pytest.mark.parametrize("n", [1, 500, 8000])
def test_num_rendered_on_a_capturing_stream(n):
    """After a small render, whose total is not read back: the call returns it
    and leaves the caller's capture whole."""
    r = _renderer()
    try:
        r.set_scene(_scene(n))
        r.set_views([_view()])
        r.render()
        exp = r.num_rendered()
        spare = torch.zeros(8, device="cuda")
        torch.cuda.synchronize()
        r.render()
        torch.cuda.synchronize()
        with _capturing(r.stream) as graph:
            spare.add_(1.0)
            got = r.num_rendered()
            spare.add_(1.0)
        assert got == exp == r.num_rendered()
        for _ in range(3):
            graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(spare, torch.full_like(spare, 6.0))
    finally:
        r.close()


def test_num_rendered_after_a_change_of_stream():
    """The total of a small render is there for a context that has gone on to
    another stream, also while that one is being captured, and after the workspace
    has been given back."""
    sc, views = _scene(700), [_view(20.0)]
    _, _, exp = _fresh(sc, views, torch.ones(40 * 33, device="cuda"))
    r = _renderer()
    try:
        r.set_scene(sc)
        r.set_views(views)
        other, spare = torch.cuda.Stream(), torch.zeros(8, device="cuda")
        torch.cuda.synchronize()
        r.render()
        binding.ddgs_set_stream(r.ctx, other.cuda_stream)
        with _capturing(other):
            spare.add_(1.0)
            got = r.num_rendered()
        binding.ddgs_set_stream(r.ctx, r.stream.cuda_stream)
        assert got == exp
        r.render()
        torch.cuda.synchronize()
        r.set_workspace(None)
        assert r.num_rendered() == exp
    finally:
        r.close()


def test_backward_of_a_replay_after_a_smaller_plain_render():
    """A plain render of fewer entries between the capture and a replay: a plain
    backward behind the replay still covers all of the replay's work items."""
    sc, near = _scene(9000), _view(10.0, 60, 52)
    pose = near.pose.copy()
    pose[0, 3] += 60.0  # most of the model beside the detector
    aside = synth.view(60, 52, 0.9, 1000.0, 600.0, 10.0, pose=pose)
    wt = torch.cos(torch.arange(60 * 52, device="cuda", dtype=torch.float32))  # (not the step's own)
    r = _renderer()
    try:
        r.set_options(split=16)
        r.set_scene(sc)
        r.set_views([near])
        r.render()
        need = r.num_rendered()
        exp = {k: v.clone() for k, v in r.backward(wt).items()}
        torch.cuda.synchronize()
        s = _capture(r, 0)
        r.set_views([aside])
        r.render()
        assert r.num_rendered() < need // 2
        r.set_views([near])
        torch.cuda.synchronize()
        binding.ddgs_step_launch(r.ctx)
        assert r.check_step() == 0 and s["img"].any()
        for g in s["grads"].values():
            g.zero_()
        torch.cuda.synchronize()
        got = r.backward(wt)
        torch.cuda.synchronize()
        for k in exp:
            assert torch.equal(got[k], exp[k]), k
    finally:
        r.close()
