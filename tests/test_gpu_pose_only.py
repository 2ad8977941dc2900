"""The pose-only projection backward (registration) has an instance of its own,
which reads a view ahead and deals the views to several blocks: its pose
gradients equal those of the full backward to the bit, over the model variants,
view counts on both sides of a block's, tiles per Gaussian on both sides of what
is read ahead, and a partial last block."""
from dataclasses import replace

import numpy as np
import pytest

from gpu_common import make_renderer
from paper_2406_02518_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,V,k,L,kind,std", [
    (1, 1, 8, 1, "mixed", 1.0), (255, 2, 8, 1, "mixed", 1.0), (257, 3, 16, 3, "dir", 2.0),
    (600, 33, 16, 3, "mixed", 0.3), (600, 70, 8, 1, "iso", 1.0), (1500, 5, 32, 3, "entangled", 3.0),
    (900, 31, 16, 3, "entangled", 0.6)])
def test_pose_only_equals_the_full_backward(n, V, k, L, kind, std):
    sc = synth.random_scene(41 + n + V, n, k=k, L=L, extent=18.0, std_range=(0.5 * std, 1.5 * std),
                            iso_fraction={"mixed": 0.8, "dir": 0.0, "iso": 1.0, "entangled": 0.0}[kind])
    if kind == "entangled":
        sc = replace(sc, n_iso=0, entangled=True)
    views = [synth.view(44 - (3 * j) % 4, 36, 0.9, 1000.0, 600.0, 11.0 * j) for j in range(V)]
    r = make_renderer()
    try:
        r.set_options(tile_w=8, tile_h=8, split=64)
        r.set_scene(sc)
        r.set_views(views)
        img = r.render()
        dl = torch.sin(torch.arange(img.numel(), device="cuda", dtype=torch.float32))
        full = r.backward(dl)["dpose"].cpu().numpy()
        pose = r.backward(dl, which=("dpose",))["dpose"].cpu().numpy()
        assert n == 1 or np.abs(full).max() > 0  # (one Gaussian may miss the detector)
        np.testing.assert_array_equal(pose, full)
    finally:
        r.close()
