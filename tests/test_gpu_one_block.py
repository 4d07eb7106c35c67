"""Reductions and scans that one block takes in one launch, around the sizes
at which the other forms take over, and captures of sizes not run before."""

import numpy as np
import pytest

from gpu_util import dev_array, host_bits, need_gpu, torch
import paper_1304_5553_amd as hm

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return need_gpu()


@pytest.mark.parametrize("fmt,bytes_per,limit", [("int", 4, 65536), ("fp8_e4m3", 1, 65536), ("float4", 48, 10922)])
@pytest.mark.parametrize("calls", [False, True])
def test_reduce_hands_over(dev, fmt, bytes_per, limit, calls):
    """Sums of small integers are exact in every order.  float4: twelve float
    arrays, 48 bytes per index, so the byte limit comes first."""
    arrays = 12 if fmt == "float4" else 1
    ctype = "float" if fmt == "float4" else fmt
    sig = "float: " + ", ".join(f"const {ctype} *a{k}" for k in range(arrays))
    expr = " + ".join(f"a{k}[i]" for k in range(arrays))
    above = limit + 1
    if calls:            # one block of the general geometry still covers up to 16 KiB per array
        expr, limit, above = f"floorf({expr})", min(limit, 4096), 20000
    h = hm.compile(expr, sig, name="oneb")
    for n in (1, 63, 1025, limit, above):
        for offset in (0, 1):
            vals = np.random.default_rng(n).integers(0, 3, (arrays, n + offset))
            dts = {"int": torch.int32, "fp8_e4m3": torch.float8_e4m3fn, "float4": torch.float32}
            xs = [torch.from_numpy(v.astype(np.float32)).to(dts[fmt]).to(dev)[offset:] for v in vals]
            out = torch.full((2,), 7.0, device=dev)
            hm.reduce(h, None, "a+b", "0", n, xs, out)
            assert out.tolist() == [float(vals[:, offset:].sum()), 7.0]
            assert len(h.last_symbols()) == (1 if n <= limit else 2), n


def test_maximum_of_nan_infinity_and_lowest(dev):
    h = hm.compile("x[i]", "float: const float *x", name="oneb")
    lowest = np.finfo(np.float32).min
    for vals in ([-np.inf] * 5, [lowest] * 65, [1.0, np.nan, 3.0], [np.inf, -np.inf]):
        out = torch.empty((), device=dev)
        hm.reduce(h, None, "max(a,b)", "-INFINITY", len(vals), [dev_array(np.array(vals, np.float32))], out)
        assert np.array_equal(host_bits(out), np.max(np.array(vals, np.float32)), equal_nan=True)


@pytest.mark.parametrize("first,then", [(100, 1 << 20), (1 << 20, 100), (100, 9 << 20), (9 << 20, 100000)])
def test_capture_of_another_size(dev, first, then):
    """A capture needs only that the operation has run once, at any size."""
    st = torch.cuda.Stream()
    h = hm.compile("k[i]", "long: const int *k", name=f"cap{first}_{then}")
    vals = np.random.default_rng(1).integers(-9, 9, max(first, then)).astype(np.int32)
    k = dev_array(vals)
    out, sc = torch.empty((), dtype=torch.int64, device=dev), torch.empty(max(first, then), dtype=torch.int64, device=dev)
    ws = torch.empty(hm.scan_workspace_bytes(h, max(first, then)), dtype=torch.uint8, device=dev)
    torch.cuda.synchronize()

    def run(n):
        hm.reduce(h, None, "a+b", "0", n, [k], out, stream=st, workspace_buf=ws)
        hm.scan(h, "a+b", "0", n, [k], sc, stream=st, workspace_buf=ws)
    run(first)
    g = hm.Graph()
    with g.capture(st):
        run(then)
    for _ in range(3):
        out.zero_(), sc.zero_()
        torch.cuda.synchronize()
        g.launch(st)
        torch.cuda.synchronize()
        assert out.item() == vals[:then].sum()
        assert np.array_equal(host_bits(sc[:then]), np.cumsum(vals[:then], dtype=np.int64))
