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


@pytest.mark.parametrize("nx,ny", [((1 << 30) + 3, 1), (1, (1 << 31) + 1001), ((1 << 30) + 77, 2)])
def test_sides_beyond_two_to_the_30(nx, ny):
    """One iteration, at places on both sides of each power of two and the ends."""
    dev = need_gpu()
    n, part = nx * ny, 1 << 28
    b = torch.rand(n, device=dev) - 0.25
    s = hcg.PoissonCG(nx, ny, device=dev)
    s.solve(b, 1)

    def rows(lo, hi):
        """(A b)[lo:hi] in float64."""
        k = torch.arange(lo, hi, device=dev)
        g = lambda at, ok: torch.where(ok, b[at.clamp(0, n - 1)].double(), 0.0)   # noqa: E731
        col = k % nx
        return (4 * b[lo:hi].double() - g(k - 1, col > 0) - g(k + 1, col < nx - 1)
                - g(k - nx, k >= nx) - g(k + nx, k < n - nx))
    rr = sum((b[lo:lo + part].double() ** 2).sum().item() for lo in range(0, n, part))
    pq = sum((b[lo:min(lo + part, n)].double() * rows(lo, min(lo + part, n))).sum().item() for lo in range(0, n, part))
    alpha = rr / pq
    at = {0, n - 4096, nx - 2048 if nx > 4096 else 0}
    at |= {p - 2048 for p in (1 << 29, 1 << 30, 1 << 31) if p + 2048 < n}
    for lo in sorted(at):
        lo = min(max(0, lo), n - 4096)
        q, v = rows(lo, lo + 4096), b[lo:lo + 4096].double()
        assert (s.q[lo:lo + 4096].double() - q).abs().max().item() <= 4 * U24 * 8
        assert (s.x[lo:lo + 4096].double() - alpha * v).abs().max().item() <= 4 * U24 * alpha
        assert (s.r[lo:lo + 4096].double() - (v - alpha * q)).abs().max().item() <= 4 * U24 * (1 + 8 * alpha)
