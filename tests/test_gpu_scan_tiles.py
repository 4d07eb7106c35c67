"""GPU parity of the scan's tile forms at the sizes where they change hands:
one tile, tile totals and rescan, and the one-pass form (tiles publish their
totals), around tile, group (64 tiles) and supergroup (64 groups) edges."""

import numpy as np
import pytest

from gpu_util import dev_array, host_bits, need_gpu, torch
import oracle
import paper_1304_5553_amd as hm

pytestmark = pytest.mark.gpu

U24 = 2.0 ** -24
# tiles of 64 elements (one wave, one element per lane): 768 tiles is the last
# size of the totals-and-rescan form
TINY = {"block": 64, "items_per_thread": 1, "vec": 1}
FOLD = 768 * 64


@pytest.fixture(scope="module")
def dev():
    return need_gpu()


def tag(h):
    return h.last_symbols()[0].split("_")[-2]


def check_int(dev, n, config, exclusive, offset=0, out_offset=0, ws=None):
    rng = np.random.default_rng(n + offset)
    base = rng.integers(-(1 << 20), 1 << 20, n + 8).astype(np.int32)
    h = hm.compile("k[i]", "long: const int *k", name="scant")
    buf = torch.full((n + out_offset + 1,), 7, dtype=torch.int64, device=dev)
    hm.scan(h, "a+b", "0", n, [dev_array(base)[offset:offset + n]], buf[out_offset:out_offset + n],
            exclusive=exclusive, config=config, workspace_buf=ws)
    got = host_bits(buf)
    want = oracle.scan("long: const int *k", "k[i]", "a+b", "0", n, [base[offset:offset + n]],
                       exclusive=exclusive).values
    assert np.array_equal(got[out_offset:out_offset + n], want)
    assert (got[:out_offset] == 7).all() and got[out_offset + n] == 7
    return tag(h)


@pytest.mark.parametrize("n,config,want", [
    (16383, None, "sc1"), (16384, None, "sc1"), (16385, None, "scd"),
    (512 * 4096, None, "scd"), (512 * 4096 + 1, None, "scd"),
    (768 * 8192, None, "scd"), (768 * 8192 + 1, None, "scl"),
    (64, TINY, "sc1"), (65, TINY, "scd"), (FOLD, TINY, "scd"), (FOLD + 1, TINY, "scl"),
    (64 * 64 * 64, TINY, "scl"), (64 * 64 * 64 + 1, TINY, "scl"), (64 * 64 * 64 + 64 * 64 + 1, TINY, "scl")])
@pytest.mark.parametrize("exclusive", [False, True])
def test_tile_edges(dev, n, config, want, exclusive):
    assert check_int(dev, n, config, exclusive) == want


@pytest.mark.parametrize("offset,out_offset", [(1, 0), (1, 1), (2, 1), (3, 0)])
@pytest.mark.parametrize("n", [5, 16385, 768 * 8192 + 5])
def test_misaligned_heads(dev, n, offset, out_offset):
    check_int(dev, n, None, True, offset, out_offset)


def test_more_than_64_supergroups(dev):
    """64^3 tiles and a few: the fold over supergroups takes a second round
    (a workspace above the minimum lets the tiles stay small)."""
    n = 64 * (64 ** 3 + 130)
    ws = torch.full((8 << 20,), 255, dtype=torch.uint8, device=dev)
    assert check_int(dev, n, TINY, False, ws=ws) == "scl"


@pytest.mark.parametrize("n", [FOLD + 1, 64 ** 3 + 77])
def test_float_one_pass(dev, n):
    """D: lane prefix V, wave scan 6, sub-tile chain U, wave totals 6, three
    folds of 6 (tiles, groups, supergroups), five joins."""
    rng = np.random.default_rng(n)
    x = rng.uniform(-1, 1, n).astype(np.float32)
    sig = "float: const float *x"
    h = hm.compile("x[i]", sig, name="scant")
    out, again = torch.empty(n, device=dev), torch.empty(n, device=dev)
    hm.scan(h, "a+b", "0", n, [dev_array(x)], out, config=TINY)
    assert tag(h) == "scl"
    hm.scan(h, "a+b", "0", n, [dev_array(x)], again, config=TINY)
    assert torch.equal(out, again)                           # whichever tile ran first
    r = oracle.scan(sig, "x[i]", "a+b", "0", n, [x])
    d = 1 + 6 + 1 + 6 + 3 * 6 + 5
    tol = d * U24 * r.abs_prefix + 2 * r.err_prefix + 1e-30
    assert (np.abs(host_bits(out).astype(np.float64) - r.values) <= tol).all()


def test_one_pass_graph_replays(dev):
    """Replays of a captured one-pass scan clear its counters themselves."""
    n = FOLD + 1
    st = torch.cuda.Stream()
    h = hm.compile("k[i]", "long: const int *k", name="scant")
    k = torch.zeros(n, dtype=torch.int32, device=dev)
    out = torch.empty(n, dtype=torch.int64, device=dev)
    ws = torch.empty(hm.scan_workspace_bytes(h, n), dtype=torch.uint8, device=dev)
    torch.cuda.synchronize()
    hm.scan(h, "a+b", "0", n, [k], out, workspace_buf=ws, stream=st, config=TINY)
    g = hm.Graph()
    with g.capture(st):
        hm.scan(h, "a+b", "0", n, [k], out, workspace_buf=ws, stream=st, config=TINY)
    for rep in range(4):
        v = np.random.default_rng(rep).integers(-1000, 1000, n).astype(np.int32)
        k.copy_(torch.from_numpy(v))
        torch.cuda.synchronize()
        g.launch(st)
        torch.cuda.synchronize()
        assert np.array_equal(host_bits(out), np.cumsum(v, dtype=np.int64)), rep
