"""The scaled norm on both sides of the magnitudes at which its first pass's
unscaled sums stand (max |x| = 0 or in [2^-40, 2^40])."""

import numpy as np
import pytest

from gpu_util import dev_array, need_gpu, torch
import oracle
import paper_1304_5553_amd as hm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt", ["float", "bfloat16"])
@pytest.mark.parametrize("flags", [0, hm.CFG_FORCE_SCALAR])
@pytest.mark.parametrize("n", [1, 17, 70001])
def test_norm_is_the_same_at_every_scale(fmt, flags, n):
    """Scaling the data by a power of two scales the norm by it, bit for bit,
    whichever pass the sums came from (values in [0.5, 1): no scaled square
    leaves the normal range), and the unscaled norm meets the 1e-6 gate."""
    need_gpu()
    rng = np.random.default_rng(n)
    bits16 = rng.integers(0x3F00, 0x3F80, n).astype(np.uint16)        # bfloat16 in [0.5, 1)
    bits16[0] = 0x3F00                                                # largest known: n == 1 gives 0.5
    vals = (bits16.astype(np.uint32) << 16).view(np.float32)
    k = hm.compile("x[i]", f"float: const {fmt} *x")
    cfg = {"flags": flags} if flags else None
    base = None
    for e in (0, -126 + 2, -80, -41, -40, -39, -38, 38, 40, 41, 42, 80, 126):
        shifted = (vals.astype(np.float64) * 2.0 ** e).astype(np.float32)
        bits = (shifted.view(np.uint32) >> 16).astype(np.uint16)
        xd = dev_array(bits, "bfloat16") if fmt == "bfloat16" else dev_array(shifted)
        g = hm.norm2(k, n, [xd], config=cfg).item()
        assert hm.norm2(k, n, [xd], config=cfg).item() == g          # the blocks' count starts over
        if base is None:
            base = g
            o = oracle.norm2(vals.astype(np.float64))
            assert abs(g - o) <= 1e-6 * o
        assert g == base * 2.0 ** e, e


def test_replays_switch_between_the_passes():
    """One captured norm over data that need the second pass and data that do not."""
    dev = need_gpu()
    n = 300007
    base = np.random.default_rng(5).uniform(0.5, 1.0, n).astype(np.float32)
    st = torch.cuda.Stream()
    k = hm.compile("x[i]", "float: const float *x")
    x, out = dev_array(base), torch.empty((), dtype=torch.float64, device=dev)
    ws = torch.empty(hm.reduce_workspace_bytes(k, n), dtype=torch.uint8, device=dev)
    torch.cuda.synchronize()
    hm.norm2(k, n, [x], out=out, workspace_buf=ws, stream=st)
    st.synchronize()
    want = out.item()
    g = hm.Graph()
    with g.capture(st):
        hm.norm2(k, n, [x], out=out, workspace_buf=ws, stream=st)
    for e in (0, 60, 60, -60, 0, 100):
        x.copy_(torch.from_numpy((base * np.float32(2.0) ** e).astype(np.float32)))
        torch.cuda.synchronize()
        g.launch(st)
        torch.cuda.synchronize()
        assert out.item() == want * 2.0 ** e, e


@pytest.mark.parametrize("fmt,tdt", [("float", torch.float32), ("bfloat16", torch.bfloat16),
                                     ("fp8_e4m3", torch.float8_e4m3fn)])
@pytest.mark.parametrize("n", [1, 4097, 100003, 1 << 22])
def test_one_launch_equals_two(fmt, tdt, n):
    """Compensated sums and one-pass norms that fold in their own launch, and
    the captured form that does not: the same bits, whatever the workspace holds."""
    dev = need_gpu()
    x = torch.randn(n + 1, device=dev).to(tdt)[1:]
    k = hm.compile("x[i]", f"float: const {fmt} *x", name="compf")
    st = torch.cuda.Stream()
    for call in (hm.reduce_compensated, lambda *a, **kw: hm.norm2(*a, passes=1, **kw)):
        out, two = (torch.zeros((), dtype=torch.float64, device=dev) for _ in range(2))
        for fill in (0, 255):
            ws = torch.full((hm.reduce_workspace_bytes(k, n),), fill, dtype=torch.uint8, device=dev)
            torch.cuda.synchronize()
            for _ in range(3):
                out.zero_()
                torch.cuda.synchronize()
                call(k, n, [x], post_scale=0.5, out=out, workspace_buf=ws, stream=st)
                assert len(k.last_symbols()) == 1
            g = hm.Graph()
            with g.capture(st):
                call(k, n, [x], post_scale=0.5, out=two, workspace_buf=ws, stream=st)
            assert len(k.last_symbols()) == 2
            for _ in range(2):
                g.launch(st)
                torch.cuda.synchronize()
                assert two.item() == out.item() and out.item() != 0.0


@pytest.mark.parametrize("grid", [1, 2, 1024, 1025, 3000])
@pytest.mark.parametrize("flags", [0, hm.CFG_FORCE_SCALAR, hm.hipmr.CFG_NO_WAIT])
def test_second_pass_of_any_grid(grid, flags):
    """Either side of the largest grid that folds in its own launch, from a
    workspace full of anything, and with the pass needed or not in turn."""
    dev = need_gpu()
    n = 1 << 22
    base = np.random.default_rng(9).uniform(0.5, 1.0, n).astype(np.float32)
    o = oracle.norm2(base.astype(np.float64))
    k = hm.compile("x[i]", "float: const float *x")
    ws = torch.full((hm.reduce_workspace_bytes(k, n),), 255, dtype=torch.uint8, device=dev)
    first = None
    for e in (0, 60, 60, -60, 0, 100):
        x = dev_array((base * np.float32(2.0) ** e).astype(np.float32))
        g = hm.norm2(k, n, [x], workspace_buf=ws, config={"grid": grid, "block": 64, "flags": flags}).item() / 2.0 ** e
        assert len(k.last_symbols()) == (2 if grid <= 1024 else 3)
        first = g if first is None else first
        assert g == first and abs(g - o) <= 1e-6 * o


@pytest.mark.parametrize("top", [-40, -39, 0, 39])
@pytest.mark.parametrize("span", [24, 40, 86])
def test_magnitudes_far_below_the_largest(top, span):
    """Values over many binades under a maximum whose unscaled squares stand:
    those below 2^-63 have subnormal squares there.  The 1e-6 gate."""
    need_gpu()
    n = 1 << 20
    rng = np.random.default_rng(span + top + 100)
    x = (rng.uniform(1.0, 2.0, n) * 2.0 ** rng.integers(top - span, top, n)).astype(np.float32)
    x[7] = np.float32(2.0) ** top
    k = hm.compile("x[i]", "float: const float *x")
    o = oracle.norm2(x.astype(np.float64))
    assert abs(hm.norm2(k, n, [dev_array(x)]).item() - o) <= 1e-6 * o


@pytest.mark.parametrize("first,then", [(5000, 1 << 20), (1 << 20, 5000)])
def test_capture_across_the_grids(first, then):
    """A geometry whose grid is above 1024 blocks for one size and below for
    the other: after a run at one, a capture of the other finds its kernels."""
    dev = need_gpu()
    cfg = {"block": 64, "blocks_per_cu": 32}
    base = np.random.default_rng(11).uniform(0.5, 1.0, 1 << 20).astype(np.float32)
    k = hm.compile("x[i]", "float: const float *x", name=f"normcap{first}")
    x, out = dev_array(base), torch.empty((), dtype=torch.float64, device=dev)
    ws = torch.empty(hm.reduce_workspace_bytes(k, 1 << 20), dtype=torch.uint8, device=dev)
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    hm.norm2(k, first, [x], out=out, workspace_buf=ws, stream=st, config=cfg)
    g = hm.Graph()
    with g.capture(st):
        hm.norm2(k, then, [x], out=out, workspace_buf=ws, stream=st, config=cfg)
    for e in (0, 60, 0):
        x.copy_(torch.from_numpy((base * np.float32(2.0) ** e).astype(np.float32)))
        torch.cuda.synchronize()
        g.launch(st)
        torch.cuda.synchronize()
        o = oracle.norm2(base[:then].astype(np.float64)) * 2.0 ** e
        assert abs(out.item() - o) <= 1e-6 * o
