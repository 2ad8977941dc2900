"""The chunked raster kernels for every tile shape: the forward with an entry
list per 4 x 4 cell against the unculled forward (bit for bit), and the
backward with a list per 8 x 8 part against the oracle, at chunk sizes around
the batches of 64, 128 and 256 entries, on ragged detectors, and behind
stacks so opaque that the transmittance underflows."""
import numpy as np
import pytest

from gpu_common import make_renderer, rel_l2, unique_pixels
from oracle import ref
from paper_2406_02518_amd import binding, synth
from test_gpu_edge import GROUPS, TOL, _opaque_scene, _parity

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [(16, 16), (16, 8), (32, 8), (8, 8)]


@pytest.fixture(scope="module")
def R():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    r = make_renderer()
    yield r
    r.close()


@pytest.mark.parametrize("tw,th", SHAPES)
@pytest.mark.parametrize("split", [1, 15, 130, 256, 700])
def test_cell_lists_equal_the_unculled_forward(R, tw, th, split):
    sc = synth.random_scene(43, 2500, k=8, L=1, extent=6.0, std_range=(0.1, 1.5), alpha_range=(0.05, 0.99))
    R.set_scene(sc)
    R.set_views([synth.view(75, 41, 0.3, 1000.0, 600.0, 20.0), synth.view(5, 3, 4.0, 1000.0, 550.0, 200.0)])
    try:
        R.set_options(tile_w=tw, tile_h=th, split=split)
        img = R.render().cpu().numpy()
        binding.ddgs_debug_count_pairs(R.ctx, 1)
        full = R.render().cpu().numpy()
        np.testing.assert_array_equal(img, full)
        assert np.abs(img).max() > 0
    finally:
        binding.ddgs_debug_count_pairs(R.ctx, 0)
        R.set_options(tile_w=16, tile_h=16, split=256)


@pytest.mark.parametrize("tw,th", SHAPES)
@pytest.mark.parametrize("split", [3, 128, 256])
def test_part_lists_backward_matches_oracle(R, tw, th, split):
    """1e-4 relative L2 in every group, as everywhere (float32 against the
    oracle); opacities on both sides of sigma_max / 2."""
    v = synth.view(61, 43, 0.5, 1000.0, 600.0, 20.0)
    try:
        R.set_options(tile_w=tw, tile_h=th, split=split)
        _parity(R, _opaque_scene(seed=21, n=400), v, None, seed=3)
        _parity(R, synth.random_scene(22, 900, k=8, L=2, extent=14.0, std_range=(0.1, 2.0)), v, None, seed=4)
    finally:
        R.set_options(tile_w=16, tile_h=16, split=256)


@pytest.mark.parametrize("tw,th", SHAPES)
def test_gradients_behind_opaque_stacks(R, tw, th):
    """4000 clamped Gaussians over each other: T passes below the smallest
    float32, gradients stay finite and those of the front agree with the oracle."""
    sc = _opaque_scene(seed=31, n=4000)
    sc.opacity_logit[:] = np.float32(6.0)
    v = synth.view(32, 32, 0.6, 1000.0, 600.0, 20.0)
    try:
        R.set_options(tile_w=tw, tile_h=th, split=256)
        R.set_scene(sc)
        R.set_views([v])
        pix = unique_pixels(sc, [v], ref.all_pixels([v]))
        lin = pix[:, 2] * v.W + pix[:, 1]
        assert len(pix) > 100
        img = R.render().cpu().numpy().astype(np.float64)
        assert np.isfinite(img).all()
        assert rel_l2(img[lin], ref.render(sc, [v])[0].ravel()[lin]) < TOL
        w = np.random.default_rng(5).normal(size=len(pix))
        dl = np.zeros(v.W * v.H, np.float32)
        dl[lin] = w
        g = R.backward(torch.from_numpy(dl).cuda())
        torch.cuda.synchronize()
        o = ref.backward(sc, [v], pix, dl[lin].astype(np.float64))
        for k in GROUPS:
            assert rel_l2(g[k].cpu().numpy(), o[k]) < TOL, k
        for scale in (1.0, 1e30, 1e-30):
            g = R.backward(torch.full((32 * 32,), scale, device="cuda"))
            torch.cuda.synchronize()
            for k, x in g.items():
                assert torch.isfinite(x).all(), (k, scale)
    finally:
        R.set_options(tile_w=16, tile_h=16, split=256)


@pytest.mark.parametrize("n", [1, 2, 2560, 2561, 7168, 7169, 14336, 14337])
def test_tile_order_around_the_sort_sizes(R, n):
    """One tile that every Gaussian reaches, at the lengths where the per-tile
    sort changes its instance: the list is in (depth key, index) order."""
    sc = synth.random_scene(51, n, k=8, L=1, extent=0.4, std_range=(2.0, 3.0), alpha_range=(0.001, 0.01))
    sc.mean[:, 1::7] = sc.mean[:, 0::7][:, :sc.mean[:, 1::7].shape[1]]  # equal depths: ties go by index
    R.set_scene(sc)
    R.set_views([synth.view(8, 8, 1.0, 1000.0, 600.0, 0.0)])
    R.render()
    assert R.num_rendered() == n
    zk = R.debug(binding.DBG_DEPTH_KEYS, np.uint32, n)
    vals = R.debug(binding.DBG_TILE_VALS, np.uint32, n)
    np.testing.assert_array_equal(vals, np.lexsort((np.arange(n), zk)))


@pytest.mark.parametrize("split", [16, 256])
def test_a_render_that_outgrows_its_buffers(split):
    """The work items are listed by the tile scan as far as the buffers go; a
    render that needs more lists them again: same image and gradients as a
    renderer whose buffers were large enough, and the next render too."""
    small = synth.random_scene(61, 40, k=8, L=1, extent=8.0)
    large = synth.random_scene(62, 6000, k=8, L=1, extent=10.0, std_range=(0.5, 2.5))
    v = synth.view(100, 70, 0.4, 1000.0, 600.0, 10.0)
    dl = torch.randn(100 * 70, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    out = []
    for warm in ((small,), (large, large)):
        r = make_renderer(split=split)
        for s in warm:
            r.set_scene(s)
            r.set_views([v])
            r.render()
        for _ in range(2):
            r.set_scene(large)
            r.set_views([v])
            img = r.render()
            g = r.backward(dl)
            torch.cuda.synchronize()
            out.append([img.cpu().numpy()] + [g[k].cpu().numpy() for k in sorted(g)])
        r.close()
    for o in out[1:]:
        for x, y in zip(out[0], o):
            np.testing.assert_array_equal(x, y)
