"""The fused CG kernels on narrow grids, whose tiles have other shapes (128 x 8,
16 x 64, 4 x 256, 1 x 1024), at the edges of those tiles."""

import numpy as np
import pytest

from gpu_util import dev_array, host_bits, need_gpu, torch
from paper_1304_5553_amd import cg as hcg
from test_gpu_cg_fused import U24, apply_a, numpy_cg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(1, 9216), (1, 9217), (1, 20000), (9217, 1), (300007, 1), (2, 10000), (3, 8193 + 255),
                                   (4, 8448), (4, 8449), (5, 9000), (15, 8256), (16, 8256), (16, 8257), (17, 16397),
                                   (33, 8195), (70001, 2), (65537, 3), (65536, 4), (65792, 5), (65, 16400)])
@pytest.mark.parametrize("iters", [1, 3])
def test_narrow_grids(nx, ny, iters):
    """The bound of the test of the wide tiles."""
    dev = need_gpu()
    rng = np.random.default_rng(nx + ny + iters)
    b = rng.uniform(-1, 1, nx * ny).astype(np.float32)
    want, rr = numpy_cg(b, nx, ny, iters)
    s = hcg.PoissonCG(nx, ny, device=dev)
    s.solve(dev_array(b), iters)
    torch.cuda.synchronize()
    for name in ("x", "r", "p", "q"):
        got = host_bits(getattr(s, name)).astype(np.float64)
        scale = np.abs(want[name]).max() + (np.abs(b).max() if name in ("r", "p") else 0)
        assert np.abs(got - want[name]).max() <= 8 * 8 * iters * U24 * scale, name
    q = apply_a(host_bits(s.p), nx, ny)                  # one more step's operator, from the solver's own p
    s.step()
    torch.cuda.synchronize()
    assert np.abs(host_bits(s.q) - q).max() <= 2 * U24 * np.abs(q).max()


@pytest.mark.parametrize("nx,ny", [(1, 20000), (16, 9001), (70001, 3)])
def test_a_run_is_the_sum_of_its_parts(nx, ny):
    dev = need_gpu()
    b = torch.randn(nx * ny, device=dev)
    whole, parts = hcg.PoissonCG(nx, ny, device=dev), hcg.PoissonCG(nx, ny, device=dev)
    x = whole.solve(b, 7)
    parts.solve(b, 2)
    for _ in range(5):
        parts.step()
    assert torch.equal(x, parts.x) and torch.equal(whole.r, parts.r) and torch.equal(whole.p, parts.p)
