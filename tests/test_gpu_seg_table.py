"""The segmented map-reduce's tile table at the edges of its planner's rounds
(64 segments per wave step, 512 or 1024 threads) and of the forms by number
of segments, with segments of zero, one and many tiles among them."""

import numpy as np
import pytest

from gpu_util import dev_array, host_bits, need_gpu, torch
import paper_1304_5553_amd as hm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("config", [None, {"flags": hm.hipmr.CFG_SEG_GLOBAL}, {"block": 256, "blocks_per_cu": 8},
                                    {"block": 64}])
@pytest.mark.parametrize("nseg", [1, 63, 64, 65, 255, 257, 511, 513, 1025, 4095, 4096, 4097, 8191, 8192, 16385,
                                  32768, 32769, 70000])
def test_integer_segments(nseg, config):
    dev = need_gpu()
    rng = np.random.default_rng(nseg)
    lens = rng.choice([0, 1, 2, 7, 63, 64, 65, 300], nseg)
    lens[rng.integers(0, nseg, 3)] = [1024, 1025, 9000]          # one tile, two tiles, several
    off = np.concatenate([[3], 3 + np.cumsum(lens)]).astype(np.int64)
    k = rng.integers(-1000, 1000, int(off[-1]) + 5).astype(np.int32)
    h = hm.compile("k[i]", "long: const int *k", name="segt")
    out = torch.full((nseg + 1,), 7, dtype=torch.int64, device=dev)
    hm.reduce_segmented(h, "a+b", "0", dev_array(off), k.size, [dev_array(k)], out[:nseg], config=config)
    sums = np.concatenate([[0], np.cumsum(k.astype(np.int64))])
    got = host_bits(out)
    assert np.array_equal(got[:nseg], sums[off[1:]] - sums[off[:-1]]) and got[nseg] == 7


@pytest.mark.parametrize("first,then", [(9000, 20000), (9000, 40000), (40000, 9000), (4096, 8000)])
def test_capture_of_another_number_of_segments(first, then):
    dev = need_gpu()
    st = torch.cuda.Stream()
    h = hm.compile("k[i]", "long: const int *k", name=f"segc{first}_{then}")
    k = torch.ones(200000, dtype=torch.int32, device=dev)
    ws = torch.empty(hm.segmented_workspace_bytes(h, 50000, 200000), dtype=torch.uint8, device=dev)
    outs = {n: torch.zeros(n, dtype=torch.int64, device=dev) for n in (first, then)}
    offs = {n: torch.arange(0, 4 * n + 1, 4, device=dev) for n in (first, then)}
    torch.cuda.synchronize()

    def run(n):
        hm.reduce_segmented(h, "a+b", "0", offs[n], 200000, [k], outs[n], workspace_buf=ws, stream=st)
    run(first)
    g = hm.Graph()
    with g.capture(st):
        run(then)
    for rep in range(3):
        k.fill_(rep)
        torch.cuda.synchronize()
        g.launch(st)
        torch.cuda.synchronize()
        assert bool((outs[then] == 4 * rep).all())
