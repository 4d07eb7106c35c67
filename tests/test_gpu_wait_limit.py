"""Waits inside a launch that are given up (CFG_NO_WAIT gives them up at the
first look): a reduction's last block computes the missing shares itself."""

import pytest

from gpu_util import host_bits, need_gpu, torch
import paper_1304_5553_amd as hm

pytestmark = pytest.mark.gpu

NO_WAIT = {"flags": hm.hipmr.CFG_NO_WAIT}


@pytest.fixture(scope="module")
def dev():
    return need_gpu()


@pytest.mark.parametrize("mapping,args", [("x[i]", 1), ("x[i]*y[i]", 2), ("x[i] - (i >= 3 ? x[i-3] : 0.0f)", 1)])
@pytest.mark.parametrize("flags", [0, hm.CFG_FORCE_SCALAR])
@pytest.mark.parametrize("n", [65537, 300007, 1 << 23])
def test_reduction_without_waiting(dev, mapping, args, flags, n):
    """The same bits as with the wait, whatever the workspace holds."""
    xs = [torch.randn(n, device=dev) for _ in range(args)]
    h = hm.compile(mapping, "float: " + ", ".join(f"const float *{'xy'[k]}" for k in range(args)), name="nowait")
    want, out = torch.empty((), device=dev), torch.empty((), device=dev)
    hm.reduce(h, None, "a+b", "0", n, xs, want, config={"flags": flags})
    for fill in (0, 255):
        ws = torch.full((hm.reduce_workspace_bytes(h, n),), fill, dtype=torch.uint8, device=dev)
        for _ in range(3):
            out.fill_(7.0)
            hm.reduce(h, None, "a+b", "0", n, xs, out, workspace_buf=ws,
                      config={"flags": flags | hm.hipmr.CFG_NO_WAIT})
            assert len(h.last_symbols()) == 1
            assert host_bits(out).tobytes() == host_bits(want).tobytes()


@pytest.mark.parametrize("result,ctype,tdt", [("double", "double", torch.float64), ("long", "int", torch.int32),
                                              ("complex64", "complex64", torch.complex64)])
def test_other_results_without_waiting(dev, result, ctype, tdt):
    n = 1000003
    x = (torch.randint(-9, 9, (n,), dtype=tdt, device=dev) if tdt == torch.int32 else torch.randn(n, dtype=tdt, device=dev))
    h = hm.compile("x[i]", f"{result}: const {ctype} *x", name="nowait")
    want, out = (torch.zeros((), dtype=hm.torch_dtype(h.result_dtype), device=dev) for _ in range(2))
    hm.reduce(h, None, "a+b", "0", n, [x], want)
    hm.reduce(h, None, "a+b", "0", n, [x], out, config=NO_WAIT)
    assert host_bits(out).tobytes() == host_bits(want).tobytes()


@pytest.mark.parametrize("n", [65537, 1 << 23])
@pytest.mark.parametrize("fmt", ["float", "fp8_e4m3"])
def test_compensated_without_waiting(dev, n, fmt):
    x = torch.randn(n, device=dev).to(torch.float32 if fmt == "float" else torch.float8_e4m3fn)
    h = hm.compile("x[i]", f"float: const {fmt} *x", name="nowait")
    for flags in (0, hm.CFG_FORCE_SCALAR):
        for run in (hm.reduce_compensated, lambda *a, **k: hm.norm2(*a, passes=1, **k),
                    lambda *a, **k: hm.norm2(*a, passes=2, **k)):
            want = run(h, n, [x], config={"flags": flags}).item()
            assert run(h, n, [x], config={"flags": flags | hm.hipmr.CFG_NO_WAIT}).item() == want


@pytest.mark.parametrize("result,ctype,tdt", [("float", "float", torch.float32), ("double", "double", torch.float64),
                                              ("complex64", "complex64", torch.complex64), ("long", "int", torch.int32)])
@pytest.mark.parametrize("exclusive", [False, True])
def test_scan_without_waiting_says_so(dev, result, ctype, tdt, exclusive):
    """Every output is the scan's or NaN (0), and the next scan reports it, once."""
    n = (1 << 25) + 3
    x = (torch.randint(1, 9, (n,), dtype=tdt, device=dev) if tdt == torch.int32 else torch.randn(n, dtype=tdt, device=dev))
    h = hm.compile("x[i]", f"{result}: const {ctype} *x", name="nowait")
    rdt = hm.torch_dtype(h.result_dtype)
    want, out = torch.zeros(n, dtype=rdt, device=dev), torch.zeros(n, dtype=rdt, device=dev)
    hm.scan(h, "a+b", "0", n, [x], want, exclusive=exclusive)
    hm.scan(h, "a+b", "0", n, [x], out, exclusive=exclusive, config=NO_WAIT)
    torch.cuda.synchronize()
    unknown = out == 0 if rdt == torch.int64 else torch.isnan(out)
    assert torch.equal(out[~unknown], want[~unknown])
    assert 0 < unknown.sum().item() < n
    with pytest.raises(hm.HipError, match="gave up"):
        hm.scan(h, "a+b", "0", n, [x], out, exclusive=exclusive)
    hm.scan(h, "a+b", "0", n, [x], out, exclusive=exclusive)
    assert torch.equal(out, want)
