"""Gaussians hundreds to thousands of pixels long and less than one wide: the
conic's determinant cancels in float32, so the chunked kernels' cell and part
lists must widen the bounding box they take from it, or take none."""
import numpy as np
import pytest

from gpu_common import make_renderer, rel_l2
from oracle import ref
from paper_2406_02518_amd import binding, synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [(16, 16), (16, 8), (32, 8), (8, 8)]
PX_MM = 1000.0 / 0.3 / 600.0  # pixels per mm at the isocentre of the views below


@pytest.fixture(scope="module")
def R():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    r = make_renderer()
    yield r
    r.close()


def _needles(sigma_px, angle, at_px, alpha):
    """Gaussians of sigma_px by 0.05 mm in the detector plane of a view at azimuth
    0, the long axis at ``angle`` from the image's columns, the mean ``at_px`` (2, n)
    pixels from the image centre; every second one isotropic."""
    n = len(sigma_px)
    sc = synth.random_scene(7, n, k=8, L=1, iso_fraction=0.5, alpha_range=(0.1, 0.4))
    sc.mean[:] = np.stack([np.zeros(n), -at_px[0] / PX_MM, at_px[1] / PX_MM])
    sc.log_scale[:] = np.log(0.05)
    sc.log_scale[1] = np.log(sigma_px / PX_MM)
    phi = np.pi - angle  # (camera x is world -y)
    sc.quat[:] = np.stack([np.cos(phi / 2), np.sin(phi / 2), np.zeros(n), np.zeros(n)])
    sc.opacity_logit[:] = np.log(alpha / (1.0 - alpha))
    return sc


def _tips(seed, n, W, H):
    """Needles whose tips, at most 900 pixels from the mean, lie in the image: the
    rounding of d^T A d there is at most 8 2^-24 4 (900^2 / 0.6) = 2.6 in the
    cut-off's 9, so exp(-d^2 / 2) stays below 4 and, at these opacities, below the
    clamp."""
    rng = np.random.default_rng(seed)
    sigma = np.exp(rng.uniform(np.log(150.0), np.log(20000.0), n))
    angle = rng.uniform(0.0, np.pi, n)
    r = np.minimum(3.0 * sigma * rng.uniform(0.9, 1.02, n), rng.uniform(100.0, 900.0, n))
    tip = np.stack([rng.uniform(-0.4 * W, 0.4 * W, n), rng.uniform(-0.4 * H, 0.4 * H, n)])
    return _needles(sigma, angle, tip - r * np.stack([np.cos(angle), np.sin(angle)]), rng.uniform(0.05, 0.2, n))


@pytest.mark.parametrize("tw,th", SHAPES)
@pytest.mark.parametrize("split", [15, 256])
def test_cell_lists_of_needles_equal_the_unculled_forward(R, tw, th, split):
    R.set_scene(_tips(3, 400, 300, 220))
    R.set_views([synth.view(300, 220, 0.3, 1000.0, 600.0, 0.0)])
    try:
        R.set_options(tile_w=tw, tile_h=th, split=split)
        img = R.render().cpu().numpy()
        binding.ddgs_debug_count_pairs(R.ctx, 1)
        full = R.render().cpu().numpy()
        assert np.isfinite(full).all() and np.count_nonzero(full) > 1000
        np.testing.assert_array_equal(img, full)
    finally:
        binding.ddgs_debug_count_pairs(R.ctx, 0)
        R.set_options(tile_w=16, tile_h=16, split=256)


@pytest.mark.parametrize("tw,th", SHAPES)
def test_part_lists_of_needles_match_the_unchunked_backward(R, tw, th):
    """Opacity and radiosity gradients (sums over the pixels that a Gaussian
    reaches, without the conic's factors) against the kernel that runs every entry
    on every pixel of its tile."""
    R.set_scene(_tips(5, 400, 300, 220))
    R.set_views([synth.view(300, 220, 0.3, 1000.0, 600.0, 0.0)])
    dl = torch.from_numpy(np.random.default_rng(2).uniform(0.5, 1.5, 300 * 220).astype(np.float32)).cuda()
    out = []
    try:
        for split in (256, 0):
            R.set_options(tile_w=tw, tile_h=th, split=split)
            R.render()
            g = R.backward(dl)
            torch.cuda.synchronize()
            out.append({k: g[k].cpu().numpy() for k in ("dopacity_logit", "dfeat", "db_iso")})
    finally:
        R.set_options(tile_w=16, tile_h=16, split=256)
    for k, x in out[0].items():
        assert np.abs(out[1][k]).max() > 0 and rel_l2(x, out[1][k]) < 1e-4, k


@pytest.mark.parametrize("tw,th", SHAPES)
def test_needles_are_seen_where_the_oracle_sees_them(R, tw, th):
    """One needle at a time with its mean on a pixel centre, where exp(-d^2 / 2) = 1
    whatever the conic's rounding (the mean is within 1e-4 px: d^2 < 1e-7): the
    pixel's value and its opacity gradient."""
    v = synth.view(64, 48, 0.3, 1000.0, 600.0, 0.0)
    at = (37, 21)
    dl = torch.zeros(64 * 48, device="cuda")
    dl[at[1] * 64 + at[0]] = 1.0
    seen = 0
    try:
        R.set_options(tile_w=tw, tile_h=th, split=256)
        R.set_views([v])
        for j in range(48):
            sc = _needles(np.array([3000.0 + 100.0 * j]), np.array([0.2 + 0.055 * j]),
                          np.array([[at[0] + 0.5 - 32.0], [at[1] + 0.5 - 24.0]]), np.array([0.3]))
            R.set_scene(sc)
            img = R.render()
            if R.num_rendered() == 0:
                continue  # (its float32 covariance is singular: not projected)
            seen += 1
            g = R.backward(dl)
            exp = ref.render(sc, [v])[0].ravel()[at[1] * 64 + at[0]]
            o = ref.backward(sc, [v], np.array([[0, at[0], at[1]]]), np.array([1.0]))
            assert exp > 0.01
            assert abs(float(img[at[1] * 64 + at[0]]) - exp) < 1e-4 * exp, j
            assert rel_l2(g["dopacity_logit"].cpu().numpy(), o["dopacity_logit"]) < 1e-4, j
        assert seen >= 24
    finally:
        R.set_options(tile_w=16, tile_h=16, split=256)
