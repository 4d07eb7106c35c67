"""The fused CG kernels at the edges of their tiles (64 columns by 8 or 16
rows), against the same iteration in numpy: float64 arithmetic, every vector
and scalar rounded to float32 where the kernels store it."""

import numpy as np
import pytest

from gpu_util import dev_array, host_bits, need_gpu, torch
from paper_1304_5553_amd import cg as hcg

pytestmark = pytest.mark.gpu

U24 = 2.0 ** -24


@pytest.fixture(scope="module")
def dev():
    return need_gpu()


def apply_a(v, nx, ny):
    g = v.reshape(ny, nx).astype(np.float64)
    q = 4.0 * g
    q[:, 1:] -= g[:, :-1]
    q[:, :-1] -= g[:, 1:]
    q[1:] -= g[:-1]
    q[:-1] -= g[1:]
    return q.ravel()


def numpy_cg(b, nx, ny, iters):
    f = np.float32
    x, r, p = np.zeros_like(b), b.copy(), b.copy()
    rr, q = f((b.astype(np.float64) ** 2).sum()), None
    for _ in range(iters):
        q = apply_a(p, nx, ny)
        pq = f((p * q).sum())
        alpha = np.float64(rr) / np.float64(pq)
        r = (r - alpha * q).astype(f)
        new = f((r.astype(np.float64) ** 2).sum())
        x = (x + alpha * p).astype(f)
        p = (r + np.float64(new) / np.float64(rr) * p).astype(f)
        rr = new
    return dict(x=x, r=r, p=p, q=q), rr


@pytest.mark.parametrize("nx,ny", [(1, 1), (1, 9), (2, 3), (63, 8), (64, 7), (65, 17), (66, 16), (129, 33),
                                   (2113, 261)])
@pytest.mark.parametrize("iters", [1, 2, 3])
def test_tile_edges(dev, nx, ny, iters):
    """Against numpy with the same roundings: sums differ in order (FP64) and
    products in contraction, so a stored float may fall to the other side of
    a tie; one such ulp passes through A (factor 8) per iteration at most."""
    rng = np.random.default_rng(nx * ny + iters)
    b = rng.uniform(-1, 1, nx * ny).astype(np.float32)
    if nx * ny == 1:
        iters = 1                      # solved by the first iteration (0 / 0 after it)
    solver = hcg.PoissonCG(nx, ny, device=dev)
    solver.solve(dev_array(b), iters)
    torch.cuda.synchronize()
    want, rr = numpy_cg(b, nx, ny, iters)
    for name, w in want.items():
        g = host_bits(getattr(solver, name)).astype(np.float64)
        scale = np.abs(w).max() + (np.abs(b).max() if name in ("r", "p") else 0)
        assert np.abs(g - w).max() <= 8 * 8 * iters * U24 * scale, name
    assert abs(float(solver.rr.item()) - rr) <= 64 * iters * U24 * (rr + U24 * float(b @ b))


def test_runs_divide_bitwise(dev):
    """start and steps, native runs and a run from the start end in the same bits."""
    nx, ny = 200, 91
    b = dev_array(np.random.default_rng(1).uniform(-1, 1, nx * ny).astype(np.float32))
    one, two = hcg.PoissonCG(nx, ny, device=dev), hcg.PoissonCG(nx, ny, device=dev)
    one.solve(b, 7)
    two.start(b)
    for run in (1, 1, 3, 2):
        two._run(None, run)
    for name in ("x", "r", "p", "q", "s"):
        assert torch.equal(getattr(one, name), getattr(two, name)), name
    assert one.parity == two.parity == 1
