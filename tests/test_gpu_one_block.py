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
            assert len(h.last_symbols()) == 1, n
            two = torch.empty((), device=dev)                    # the general form, partials and their fold
            hm.reduce(h, None, "a+b", "0", n, xs, two, config={"block": 512})
            assert two.item() == out[0].item()


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


@pytest.mark.parametrize("result,ctype,tdt", [("float", "float", torch.float32), ("double", "double", torch.float64),
                                              ("long", "int", torch.int32), ("unsigned", "int", torch.int32),
                                              ("complex64", "complex64", torch.complex64)])
@pytest.mark.parametrize("n", [65537, 100003, 300007, 1 << 22])
def test_one_launch_equals_two(dev, result, ctype, tdt, n):
    """The launch that folds its own partials against partials and fold kernel
    (the same geometry, asked for): the same bits, from a workspace full of
    anything, call after call, and from a capture (which takes two launches)."""
    x = (torch.randint(-9, 9, (n,), dtype=torch.int32, device=dev) if tdt == torch.int32
         else torch.randn(n, dtype=tdt, device=dev))
    h = hm.compile("x[i]", f"{result}: const {ctype} *x", name="fin")
    rdt = hm.torch_dtype(h.result_dtype)
    out, two = torch.zeros((), dtype=rdt, device=dev), torch.zeros((), dtype=rdt, device=dev)
    nbytes = hm.reduce_workspace_bytes(h, n)
    cfg = {"block": 256, "items_per_thread": 4, "blocks_per_cu": 2}
    for fill in (0, 255, 17):
        ws = torch.full((nbytes,), fill, dtype=torch.uint8, device=dev)
        hm.reduce(h, None, "a+b", "0", n, [x], two, workspace_buf=ws, config=cfg)
        assert len(h.last_symbols()) == 2
        for _ in range(3):
            out.zero_()
            hm.reduce(h, None, "a+b", "0", n, [x], out, workspace_buf=ws)
            assert len(h.last_symbols()) == 1
            assert host_bits(out).tobytes() == host_bits(two).tobytes()
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    g = hm.Graph()
    with g.capture(st):
        hm.reduce(h, None, "a+b", "0", n, [x], out, workspace_buf=ws, stream=st)
    assert len(h.last_symbols()) == 2
    tg = torch.cuda.CUDAGraph()                                  # a capture the library was not told of
    with torch.cuda.graph(tg):
        hm.reduce(h, None, "a+b", "0", n, [x], out, workspace_buf=ws)
    assert len(h.last_symbols()) == 2
    for replay in (lambda: g.launch(st), tg.replay) * 3:
        x.neg_()
        torch.cuda.synchronize()
        replay()
        torch.cuda.synchronize()
        hm.reduce(h, None, "a+b", "0", n, [x], two)
        assert host_bits(out).tobytes() == host_bits(two).tobytes()
