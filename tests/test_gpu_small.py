"""Small inputs, which one workgroup bins and whose plain render does not wait
for its entry total: the same lists, images and gradients as the general
binning gives, around the limits of the rule that selects it."""
import numpy as np
import pytest

from gpu_common import make_renderer
from paper_2406_02518_amd import binding, synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _views(V, w, h):
    return [synth.view(w - (3 * j) % 4, h, 0.9, 1000.0, 600.0, 25.0 * j) for j in range(V)]


def _lists(r, sc, views, opts):
    r.set_options(**opts)
    r.set_scene(sc)
    r.set_views(views)
    img = r.render()
    dl = torch.sin(torch.arange(img.numel(), device="cuda", dtype=torch.float32))
    g = r.backward(dl)
    torch.cuda.synchronize()
    M = r.num_rendered()
    base = r.debug(binding.DBG_TILE_BASE, np.int32, len(views) + 1)
    return [img.cpu().numpy(), r.debug(binding.DBG_TILE_VALS, np.uint32, M),
            r.debug(binding.DBG_RANGES, np.uint32, 2 * int(base[-1]))] + [g[k].cpu().numpy() for k in sorted(g)]


# (the rule: n V <= 8192, up to 4096 tiles, n x tiles <= 2^18; the pairs of
# sizes sit on both sides of it, the last is beyond the entry limit)
@pytest.mark.parametrize("n,V,w,h", [(1, 1, 5, 4), (255, 3, 40, 33), (2000, 1, 64, 64), (257, 31, 24, 16),
                                     (8192, 1, 80, 80), (8193, 1, 80, 80), (2731, 3, 64, 48), (3000, 1, 300, 290)])
@pytest.mark.parametrize("opts", [dict(tile_w=16, tile_h=16, split=256), dict(tile_w=8, tile_h=8, split=64),
                                  dict(tile_w=32, tile_h=8, split=0), dict(tile_w=16, tile_h=8, split=0, persistent=1)])
def test_small_binning_equals_the_general_one(n, V, w, h, opts):
    sc = synth.random_scene(71 + n, n, k=8, L=1, extent=18.0, std_range=(0.3, 2.0))
    views = _views(V, w, h)
    a, b = make_renderer(), make_renderer()
    try:
        got = _lists(a, sc, views, opts)
        # a caller region is not grown for the small path: the general binning
        b.set_options(**opts)
        b.set_scene(sc)
        b.set_views(views)
        ws = torch.empty(b.workspace_size(max(1, got[1].size)) + (1 << 20), dtype=torch.uint8, device="cuda")
        b.set_workspace(ws)
        exp = _lists(b, sc, views, opts)
        for x, y in zip(got, exp):
            np.testing.assert_array_equal(x, y)
    finally:
        a.close()
        b.close()


@pytest.mark.parametrize("n", [900, 3000])
def test_small_captured_step_equals_the_plain_path(n):
    """Replays (with eager work between them) against the plain calls, and an
    overflow of the captured capacity."""
    sc = synth.random_scene(91, n, k=8, L=1, extent=18.0)
    views = _views(2, 48, 40)
    r = binding.Renderer(0, stream=torch.cuda.Stream())
    try:
        r.set_scene(sc)
        r.set_views(views)
        P = r.image_size()
        img, dl = torch.empty(P, device="cuda"), torch.empty(P, device="cuda")
        loss = torch.empty(2, device="cuda")
        w = torch.sin(torch.arange(P, device="cuda", dtype=torch.float32))
        grads = r.alloc_grads()

        def capture():
            with torch.cuda.stream(r.stream):
                binding.ddgs_step_capture(r.ctx, binding.LOSS_LINEAR, w.data_ptr(), 0.0, img.data_ptr(), dl.data_ptr(),
                                          loss.data_ptr(), r.grads_struct(grads))

        torch.cuda.synchronize()
        exp_img = r.render().clone()
        exp_g = {k: v.clone() for k, v in r.backward(w).items()}
        torch.cuda.synchronize()
        need = r.num_rendered()
        capture()
        for _ in range(3):
            binding.ddgs_step_launch(r.ctx)
            assert r.check_step() == 0
            torch.cuda.synchronize()
            assert torch.equal(img, exp_img)
            for k in exp_g:
                assert torch.equal(grads[k], exp_g[k]), k
            (w * 2.0).sum().item()
        r.set_options(capacity=need - 1)
        capture()
        binding.ddgs_step_launch(r.ctx)
        assert r.check_step() == 1
        capture()
        binding.ddgs_step_launch(r.ctx)
        assert r.check_step() == 0
        assert torch.equal(img, exp_img)
    finally:
        r.close()


@pytest.mark.parametrize("opts", [dict(tile_w=16, tile_h=16, split=256), dict(tile_w=8, tile_h=8, split=64),
                                  dict(tile_w=16, tile_h=8, split=0, persistent=1)])
def test_renders_after_smaller_and_larger_ones(opts):
    """A plain render scatters and sorts into the buffers that earlier renders
    sized before it knows its entry total: totals within their spare room,
    beyond it, and smaller ones again, ranges of long tiles, and more tiles than
    the one-launch scan takes, each equal to a fresh renderer's first render."""
    a = make_renderer()
    try:
        for n, w, h, V in [(9000, 60, 52, 1), (9900, 60, 52, 1), (40000, 60, 52, 1), (9000, 60, 52, 2),
                           (60000, 33, 20, 1), (60000, 1100, 1000, 1), (9000, 17, 16, 1)]:
            sc = synth.random_scene(17, n, k=4, L=1, extent=18.0, std_range=(0.3, 1.5))
            views = _views(V, w, h)
            b = make_renderer()
            got, exp = _lists(a, sc, views, opts), _lists(b, sc, views, opts)
            b.close()
            for x, y in zip(got, exp):
                np.testing.assert_array_equal(x, y)
    finally:
        a.close()


def test_groups_of_many_tiles_equal_single_views():
    """Gaussians x tiles beyond the count matrix of 1024-Gaussian groups: the
    batch's larger groups (with a partial last one) give every view the image
    and the lists that it gets alone, where the groups are the smaller ones."""
    n, opts = 200001, dict(tile_w=8, tile_h=8, split=256)
    sc = synth.random_scene(23, n, k=4, L=1, extent=60.0, std_range=(0.05, 0.3))
    views = [synth.view(1900 - 3 * j, 1880, 0.12, 1000.0, 600.0, 25.0 * j) for j in range(7)]
    tiles = [-(-v.W // 8) * -(-v.H // 8) for v in views]
    assert -(-n // 1024) * sum(tiles) > 64 << 20 > -(-n // 1024) * max(tiles)
    r = make_renderer()
    try:
        r.set_options(**opts)
        r.set_scene(sc)
        r.set_views(views)
        imgs = [x.clone() for x in r.split(r.render())]
        M = r.num_rendered()
        vals = r.debug(binding.DBG_TILE_VALS, np.uint32, M)
        at = 0
        for v, img in zip(views, imgs):
            r.set_views([v])
            assert torch.equal(r.split(r.render())[0], img)
            m = r.num_rendered()
            np.testing.assert_array_equal(r.debug(binding.DBG_TILE_VALS, np.uint32, m), vals[at:at + m])
            at += m
        assert at == M and M > n
    finally:
        r.close()


@pytest.mark.parametrize("n,w,h", [(20000, 40, 30), (60000, 24, 20), (60000, 256, 250)])
def test_long_tiles_of_few(n, w, h):
    """Long ranges among no more tiles than the card has compute units, sorted
    beside the short ones in one launch: a render that has seen the layout, and a
    captured step, against the first render (two launches); lists beyond the LDS
    (more than 14336 entries in a tile) included."""
    sc = synth.random_scene(29, n, k=4, L=1, extent=18.0, std_range=(1.0, 4.0))
    views = _views(1, w, h)
    r = binding.Renderer(0, stream=torch.cuda.Stream())
    try:
        opts = dict(tile_w=16, tile_h=16, split=256)
        first = _lists(r, sc, views, opts)
        again = _lists(r, sc, views, opts)
        for x, y in zip(again, first):
            np.testing.assert_array_equal(x, y)
        ln = first[2].reshape(-1, 2)[:, 1].astype(np.int64) - first[2].reshape(-1, 2)[:, 0]
        assert ln.size <= 256 and ln.max() > (14336 if (n, w) == (60000, 24) else 2560)
        P = r.image_size()
        img, dl, w_ = torch.empty(P, device="cuda"), torch.empty(P, device="cuda"), torch.ones(P, device="cuda")
        loss, grads = torch.empty(1, device="cuda"), r.alloc_grads()
        torch.cuda.synchronize()
        with torch.cuda.stream(r.stream):
            binding.ddgs_step_capture(r.ctx, binding.LOSS_LINEAR, w_.data_ptr(), 0.0, img.data_ptr(), dl.data_ptr(),
                                      loss.data_ptr(), r.grads_struct(grads))
        for _ in range(3):
            binding.ddgs_step_launch(r.ctx)
            assert r.check_step() == 0
            torch.cuda.synchronize()
            np.testing.assert_array_equal(img.cpu().numpy(), first[0])
    finally:
        r.close()


@pytest.mark.parametrize("n", [500, 12000])
def test_plain_render_refuses_a_capture(n):
    """A plain render reads its entry total back, at once or later, so a stream
    that is being captured is refused, and the render works again afterwards."""
    sc = synth.random_scene(31, n, k=4, L=1, extent=18.0)
    r = binding.Renderer(0, stream=torch.cuda.Stream())
    try:
        r.set_scene(sc)
        r.set_views(_views(1, 40, 33))
        torch.cuda.synchronize()
        img = r.render().clone()
        out, spare = torch.empty_like(img), torch.zeros(8, device="cuda")
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.stream(r.stream):
            graph.capture_begin(capture_error_mode="thread_local")
            spare.add_(1.0)
            with pytest.raises(binding.DDGSError):
                binding.ddgs_render(r.ctx, out.data_ptr())
            graph.capture_end()
        torch.cuda.synchronize()
        assert torch.equal(r.render(), img)
    finally:
        r.close()


def test_long_tiles_at_two_per_compute_unit():
    """Between one and two tiles per compute unit the ranges are sorted in one
    launch while none is known beyond what that launch's LDS holds: a first
    render, one that has seen the layout, then one of the same layout with a range
    beyond it, and one that knows of it, each equal to a fresh renderer's."""
    opts, views = dict(tile_w=16, tile_h=16, split=256), [synth.view(320, 310, 0.9, 1000.0, 600.0, 20.0)]
    even = synth.random_scene(37, 20000, k=4, L=1, extent=18.0, std_range=(0.5, 1.5))
    heap = synth.random_scene(38, 20000, k=4, L=1, extent=5.0, std_range=(0.5, 1.5))
    a = make_renderer()
    try:
        for sc, low, high in [(even, 2560, 7168), (even, 2560, 7168), (heap, 7168, 20001), (heap, 7168, 20001)]:
            b = make_renderer()
            got, exp = _lists(a, sc, views, opts), _lists(b, sc, views, opts)
            b.close()
            for x, y in zip(got, exp):
                np.testing.assert_array_equal(x, y)
            rg = got[2].reshape(-1, 2).astype(np.int64)
            assert rg.shape[0] == 400 and low < (rg[:, 1] - rg[:, 0]).max() <= high
    finally:
        a.close()
