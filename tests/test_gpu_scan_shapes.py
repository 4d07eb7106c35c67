"""Scan tiles by what the map holds per element, and by the caller's geometry:
a geometry asked for never makes the one-pass form's tiles smaller than its
own, nor a thread's run larger than its registers."""

import numpy as np
import pytest

from gpu_util import need_gpu, torch
import paper_1304_5553_amd as hm

pytestmark = pytest.mark.gpu

TINY = {"block": 64, "items_per_thread": 1, "vec": 1}


@pytest.fixture(scope="module")
def dev():
    return need_gpu()


def kernels(h, n, xs, out, **kw):
    hm.scan(h, "a+b", "0", n, xs, out, **kw)
    return h.last_symbols()


def test_small_tiles_asked_for(dev):
    n = (1 << 24) + 3
    x = torch.randint(0, 2, (n,), device=dev).float()            # exact sums
    h = hm.compile("x[i]", "float: const float *x", name="scshape")
    out, want = torch.empty(n, device=dev), torch.cumsum(x.double(), 0).float()
    base = kernels(h, n, [x], out)
    assert torch.equal(out, want)
    for cfg in ({"block": 64, "items_per_thread": 4}, {"block": 256}, {"items_per_thread": 1}):
        out.zero_()
        assert kernels(h, n, [x], out, config=cfg) == base, cfg
        assert torch.equal(out, want)


@pytest.mark.parametrize("n", [16384, 100003, (1 << 24) + 3])
def test_runs_longer_than_the_registers(dev, n):
    x = torch.randint(0, 2, (n,), device=dev).float()
    h = hm.compile("x[i]", "float: const float *x", name="scshape")
    out, want = torch.empty(n, device=dev), torch.cumsum(x.double(), 0).float()
    longest = kernels(h, n, [x], out, config={"block": 1024, "items_per_thread": 4, "vec": 16})
    assert torch.equal(out, want)
    out.zero_()
    assert kernels(h, n, [x], out, config={"block": 1024, "items_per_thread": 16, "vec": 16}) == longest
    assert torch.equal(out, want)


@pytest.mark.parametrize("kind", ["call", "combine", "twelve"])
@pytest.mark.parametrize("n", [1, 4096, 4097, 1 << 20, (1 << 20) + 1, 1 << 21, (1 << 21) + 1, 768 * 4096,
                               768 * 4096 + 1, 768 * 8192, 768 * 8192 + 1])
@pytest.mark.parametrize("exclusive", [False, True])
def test_edges_of_the_forms(dev, kind, n, exclusive):
    """Whole numbers: exact in any order."""
    arrays = 12 if kind == "twelve" else 1
    xs = [torch.randint(0, 2, (n,), device=dev).float() for _ in range(arrays)]
    expr = " + ".join(f"x{k}[i]" for k in range(arrays))
    h = hm.compile(f"floorf({expr})" if kind == "call" else expr,
                   "int: " + ", ".join(f"const float *x{k}" for k in range(arrays)), name="scshape")
    out = torch.full((n + 1,), 7, dtype=torch.int32, device=dev)
    hm.scan(h, "floorf(a + b)" if kind == "combine" else "a+b", "0", n, xs, out[:n], exclusive=exclusive)
    total = sum(x.double() for x in xs)
    want = torch.cumsum(total, 0)
    assert torch.equal(out[:n].double(), want - total if exclusive else want) and out[n] == 7


@pytest.mark.parametrize("tiles", [64 * 64, 64 * 64 + 1, 64 * 64 * 2 + 65])
def test_supergroups_of_tiles(dev, tiles):
    n = tiles * 8192 - 5
    k = torch.randint(-9, 9, (n,), dtype=torch.int8, device=dev)
    h = hm.compile("k[i]", "int: const char *k", name="scshape")
    out = torch.empty(n, dtype=torch.int32, device=dev)
    assert kernels(h, n, [k], out, config=TINY)[0].split("_")[-2] == "scl"
    assert torch.equal(out, torch.cumsum(k, 0, dtype=torch.int32))


def test_more_than_64_supergroups_of_tiles(dev):
    """The fold over supergroups takes a second round (the workspace holds every tile)."""
    n = (64 ** 3 + 130) * 8192
    k = torch.randint(-9, 9, (n,), dtype=torch.int8, device=dev)
    h = hm.compile("k[i]", "int: const char *k", name="scshape")
    out = torch.empty(n, dtype=torch.int32, device=dev)
    hm.scan(h, "a+b", "0", n, [k], out, config=TINY,
            workspace_buf=torch.full((8 << 20,), 255, dtype=torch.uint8, device=dev))
    carry = 0
    for lo in range(0, n, 1 << 28):
        part = torch.cumsum(k[lo:lo + (1 << 28)], 0, dtype=torch.int32) + carry
        assert torch.equal(out[lo:lo + (1 << 28)], part), lo
        carry = part[-1].item()


@pytest.mark.parametrize("exclusive", [False, True])
@pytest.mark.parametrize("flags", [0, hm.hipmr.CFG_NO_WAIT])
def test_parts_of_the_tiles_at_a_time(dev, exclusive, flags):
    """A workspace asked for at n = 1 takes any n: three launches' worth of
    tiles, each from what the one before handed on."""
    n = 2 * 64000 * 8192 + 12345
    k = torch.randint(-9, 9, (n,), dtype=torch.int8, device=dev)
    h = hm.compile("k[i]", "int: const char *k", name="scshape")
    ws = torch.full((hm.scan_workspace_bytes(h, 1),), 255, dtype=torch.uint8, device=dev)
    assert hm.scan_workspace_bytes(h, n) == ws.numel()
    out = torch.empty(n, dtype=torch.int32, device=dev)
    hm.scan(h, "a+b", "0", n, [k], out, exclusive=exclusive, workspace_buf=ws, config={**TINY, "flags": flags})
    torch.cuda.synchronize()
    carry, bad = 0, 0
    for lo in range(0, n, 1 << 28):
        v = k[lo:lo + (1 << 28)]
        part = torch.cumsum(v, 0, dtype=torch.int32) + carry
        carry = part[-1].item()
        got = out[lo:lo + (1 << 28)]
        wrong = got != (part - v if exclusive else part)
        bad += wrong.sum().item()
        assert (got[wrong] == 0).all()                # only sums that are not known, and said so
    if flags:
        with pytest.raises(hm.HipError, match="gave up"):
            hm.scan(h, "a+b", "0", 10, [k], out)
    else:
        assert bad == 0


@pytest.mark.parametrize("first,second", [({"block": 512}, None), (None, {"block": 512}),
                                          ({"items_per_thread": 8}, None), (None, {"items_per_thread": 8})])
@pytest.mark.parametrize("captured", [100, 100003, 1 << 23])
def test_capture_after_another_geometry(dev, first, second, captured):
    """A call that names what another leaves open (512 threads, 8 runs) has
    kernels of its own: after each has run once, at one size, a capture of the
    second at any size finds all it needs."""
    n = 1 << 23
    k = torch.randint(-9, 9, (n,), dtype=torch.int32, device=dev)
    tag = f"{'d' if first is None else list(first)[0][0]}{captured}"
    h = hm.compile("k[i]", "long: const int *k", name=f"scfam{tag}")
    out = torch.zeros(n, dtype=torch.int64, device=dev)
    ws = torch.empty(hm.scan_workspace_bytes(h, n), dtype=torch.uint8, device=dev)
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    for cfg in (first, second):
        hm.scan(h, "a+b", "0", 300007, [k], out, workspace_buf=ws, stream=st, config=cfg)
    g = hm.Graph()
    with g.capture(st):
        hm.scan(h, "a+b", "0", captured, [k], out, workspace_buf=ws, stream=st, config=second)
    for _ in range(3):
        out.zero_()
        torch.cuda.synchronize()
        g.launch(st)
        torch.cuda.synchronize()
        assert torch.equal(out[:captured], torch.cumsum(k[:captured], 0, dtype=torch.int64))
