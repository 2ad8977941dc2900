"""Which inputs one workgroup bins: bounded by their entries, as far as they are
known, and by their pairs (fewer in a captured step); the same results on both
sides of every limit."""
import numpy as np
import pytest

from gpu_common import make_renderer
from paper_2406_02518_amd import binding, synth
from test_gpu_small import _lists, _views

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

OPTS = dict(tile_w=16, tile_h=16, split=256)


def _capture(r, V):
    P = r.image_size()
    s = [torch.empty(P, device="cuda"), torch.empty(P, device="cuda"), torch.empty(V, device="cuda"), r.alloc_grads(),
         torch.sin(torch.arange(P, device="cuda", dtype=torch.float32))]
    torch.cuda.synchronize()
    with torch.cuda.stream(r.stream):
        binding.ddgs_step_capture(r.ctx, binding.LOSS_LINEAR, s[4].data_ptr(), 0.0, s[0].data_ptr(), s[1].data_ptr(),
                                  s[2].data_ptr(), r.grads_struct(s[3]))
    return s


def test_a_step_of_many_entries_is_not_binned_by_one_workgroup():
    """8000 Gaussians on 4096 tiles with some 10^7 entries take no longer than 8200
    (per entry, with half as much to spare): one workgroup took 2.4 times as long."""
    v = synth.view(1024, 1024, 80.0 / 1024, 1000.0, 600.0, 10.0)
    per_entry = []
    for n in (8000, 8200):
        r = binding.Renderer(0, stream=torch.cuda.Stream())
        try:
            r.set_options(**OPTS)
            r.set_scene(synth.random_scene(5, n, k=8, L=1, extent=20.0, std_range=(4.0, 6.0), alpha_range=(0.01, 0.1)))
            r.set_views([v])
            r.render()
            M = r.num_rendered()
            keep = _capture(r, 1)
            ts = []
            for _ in range(6):
                a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                a.record(r.stream)
                binding.ddgs_step_launch(r.ctx)
                b.record(r.stream)
                torch.cuda.synchronize()
                ts.append(a.elapsed_time(b))
            assert r.check_step() == 0 and keep[0].any()
            per_entry.append(min(ts) / M)
        finally:
            r.close()
    assert per_entry[0] < 1.5 * per_entry[1]


@pytest.mark.parametrize("n,V,w,h", [(4096, 1, 64, 64), (4097, 1, 64, 64), (1365, 3, 48, 40), (132, 31, 24, 16),
                                     (2048, 1, 60, 50), (1, 1, 5, 4)])
def test_both_sides_of_the_pair_limits(n, V, w, h):
    """Plain renders, the second one with its total known, and a captured step,
    against a caller region (not grown for the small path: the general binning)."""
    sc = synth.random_scene(71 + n, n, k=8, L=1, extent=18.0, std_range=(0.3, 2.0))
    views = _views(V, w, h)
    a, b = binding.Renderer(0, stream=torch.cuda.Stream()), make_renderer()
    try:
        first, again = _lists(a, sc, views, OPTS), _lists(a, sc, views, OPTS)
        b.set_options(**OPTS)
        b.set_scene(sc)
        b.set_views(views)
        ws = torch.empty(b.workspace_size(max(1, first[1].size)) + (1 << 20), dtype=torch.uint8, device="cuda")
        b.set_workspace(ws)
        exp = _lists(b, sc, views, OPTS)
        for x, y, z in zip(first, again, exp):
            np.testing.assert_array_equal(x, z)
            np.testing.assert_array_equal(y, z)
        s = _capture(a, V)
        for _ in range(3):
            binding.ddgs_step_launch(a.ctx)
            assert a.check_step() == 0
            torch.cuda.synchronize()
            np.testing.assert_array_equal(s[0].cpu().numpy(), exp[0])
            s[4].mul(2.0).sum().item()
    finally:
        a.close()
        b.close()


def test_totals_that_grow_and_shrink():
    """One layout whose total passes the limit and falls below it again, read or not
    read between the renders: each render equals a fresh renderer's."""
    views = _views(1, 128, 128)
    scenes = [synth.random_scene(s, 2000, k=4, L=1, extent=18.0, std_range=(std, 1.1 * std))
              for s, std in ((1, 0.5), (2, 6.0), (3, 6.0), (4, 0.5), (5, 0.5), (6, 0.4), (7, 3.0), (8, 0.5))]
    exp, totals = [], []
    for sc in scenes:
        f = make_renderer()
        f.set_options(**OPTS)
        f.set_scene(sc)
        f.set_views(views)
        exp.append(f.render().cpu().numpy())
        totals.append(f.num_rendered())
        f.close()
    assert max(totals) > 16384 > min(totals)
    r = make_renderer()
    try:
        r.set_options(**OPTS)
        for read in (True, False):
            for sc, e, t in zip(scenes, exp, totals):
                r.set_scene(sc)
                r.set_views(views)
                img = r.render()
                if read:
                    assert r.num_rendered() == t
                else:
                    torch.cuda.synchronize()
                np.testing.assert_array_equal(img.cpu().numpy(), e)
    finally:
        r.close()
