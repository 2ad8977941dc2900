"""Dual sampling where scratch memory is short."""
import numpy as np
import pytest

from paper_2406_02518_amd import binding, rads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("shape,n2,room", [((16, 16, 16), 20000, 400000), ((16, 16, 16), 20000, 8 << 20),
                                           ((70, 60, 50), 5000, 24 << 20)])
def test_neighbour_scales_in_a_caller_region(shape, n2, room):
    """A region without room for the neighbour grid (or a volume so small that the
    grid would take more of it than the volume's own scratch once did) serves the
    call all the same, with the same points and scales."""
    hu = torch.from_numpy(np.random.default_rng(3).uniform(-1000.0, 1500.0, shape).astype(np.float32)).cuda()
    r = binding.Renderer(0, stream=torch.cuda.Stream())
    try:
        torch.cuda.synchronize()
        exp = rads.sample(r, hu, (1.0, 1.0, 1.0), (0.0, 0.0, 0.0), n1=1500, n2=n2, seed=4)
        torch.cuda.synchronize()
        assert exp[0].shape[1] > 4096
        ws = torch.empty(room, dtype=torch.uint8, device="cuda")
        r.set_workspace(ws)
        for _ in range(2):
            got = rads.sample(r, hu, (1.0, 1.0, 1.0), (0.0, 0.0, 0.0), n1=1500, n2=n2, seed=4)
            torch.cuda.synchronize()
            assert torch.equal(got[0], exp[0]) and torch.equal(got[1], exp[1]) and got[2] == exp[2]
    finally:
        r.close()
