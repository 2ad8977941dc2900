"""Dual sampling where scratch memory is short, and from keys that do not fill
their 32 bits."""
import ctypes
import time

import numpy as np
import pytest

from oracle import rads_ref
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


def _keys(kind, M, rng):
    if kind == "permutation":
        return rng.permutation(M).astype(np.uint32)
    if kind == "15 bits":  # many ties
        return rng.integers(0, 1 << 15, M, dtype=np.uint32)
    if kind == "interval":  # a narrow one far from zero, across a power of two
        return (0x3FFFF000 + rng.integers(0, 1 << 20, M, dtype=np.uint64)).astype(np.uint32)
    if kind == "floats":
        return rng.random(M, dtype=np.float32).view(np.uint32)
    if kind == "two values":
        return np.where(rng.random(M) < 0.5, 7, 8).astype(np.uint32)
    k = (rng.random(M) ** 24 * 4294967295.0).astype(np.uint64)  # most of them small
    return np.minimum(k, 0xFFFFFFFF).astype(np.uint32)


@pytest.mark.parametrize("kind", ["permutation", "15 bits", "interval", "floats", "two values", "skewed"])
@pytest.mark.parametrize("shape", [(3, 4, 5), (12, 13, 14), (45, 46, 47)])
def test_key_subsample_of_narrow_ranges(kind, shape):
    """The points of the smallest keys in key order, ties by edge order, for keys that
    do not fill the 32 bits (and one that fills them unevenly)."""
    rng = np.random.default_rng(sum(shape))
    hu = rng.uniform(-1000.0, 1500.0, shape).astype(np.float32)
    t = torch.from_numpy(hu).cuda()
    f3 = ctypes.c_float * 3
    vol = binding.ddgs_volume(shape[2], shape[1], shape[0], f3(1.0, 1.0, 1.0), f3(0.0, 0.0, 0.0), t.data_ptr())
    r = binding.Renderer(0)
    try:
        level, M, _ = binding.ddgs_rads_prepare(r.ctx, vol)
        pmc, _ = rads_ref.crossings(hu, level, (1.0, 1.0, 1.0), (0.0, 0.0, 0.0))
        assert M == len(pmc)
        keys = _keys(kind, M, rng)
        order = np.lexsort((np.arange(M), keys))
        kd = torch.from_numpy(keys.view(np.int32)).cuda()
        for n1 in (1, 1700, M):
            n = min(n1, M)
            pts = torch.empty((3, n), device="cuda")
            assert binding.ddgs_rads_sample(r.ctx, n1, kd.data_ptr(), 0, None, pts.data_ptr(), None) == n
            torch.cuda.synchronize()
            np.testing.assert_allclose(pts.cpu().numpy().T, pmc[order[:n]], rtol=0, atol=2e-4)
    finally:
        r.close()


def test_a_permutation_costs_what_random_keys_do():
    """126 thousand consecutive keys in random order against random 32-bit ones: one
    workgroup had to sort them all and took 29 times as long (2 allowed here)."""
    shape = (64, 64, 32)
    hu = torch.from_numpy(np.random.default_rng(1).uniform(0.0, 1.0, shape).astype(np.float32)).cuda()
    f3 = ctypes.c_float * 3
    vol = binding.ddgs_volume(shape[2], shape[1], shape[0], f3(1.0, 1.0, 1.0), f3(0.0, 0.0, 0.0), hu.data_ptr())
    r = binding.Renderer(0)
    try:
        _, M, _ = binding.ddgs_rads_prepare(r.ctx, vol)
        assert 100000 < M <= 1 << 18
        pts = torch.empty((3, 15000), device="cuda")
        best = []
        for keys in (torch.randint(-(1 << 31), 1 << 31, (M,), device="cuda"), torch.randperm(M, device="cuda")):
            keys = keys.to(torch.int32)
            ts = []
            for _ in range(12):
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                binding.ddgs_rads_sample(r.ctx, 15000, keys.data_ptr(), 0, None, pts.data_ptr(), None)
                torch.cuda.synchronize()
                ts.append(time.perf_counter() - t0)
            best.append(min(ts))
        assert best[1] < 2.0 * best[0]
    finally:
        r.close()
