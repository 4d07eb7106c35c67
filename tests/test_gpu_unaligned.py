"""Arrays that share no 16-byte alignment (views shifted against each other):
the chunk kernels load them at element alignment, and agree bit for bit with
the one-element kernels (elementwise) and with the oracle (reductions)."""

import numpy as np
import pytest

from gpu_util import dev_array, host_bits, need_gpu, torch
import oracle
import paper_1304_5553_amd as hm

pytestmark = pytest.mark.gpu

SCALAR = {"flags": hm.CFG_FORCE_SCALAR}
# one element, below / at / above a chunk, a wave, a block; a ragged middle
SIZES = [1, 3, 4, 5, 17, 255, 257, 1025, 4099, 70001]


@pytest.fixture(scope="module")
def dev():
    return need_gpu()


def tag(k):
    return k.last_symbols()[0].split("_")[-2]


def values(dt, n, rng):
    if dt == torch.complex64:
        return torch.view_as_complex(torch.from_numpy(rng.uniform(-2, 2, (n, 2)).astype(np.float32)))
    if dt == torch.int32:
        return torch.from_numpy(rng.integers(-1000, 1000, n).astype(np.int32))
    return torch.from_numpy(rng.uniform(-2, 2, n).astype(np.float32)).to(dt)


EW = [("z[i] = 2.5f*x[i] - 0.5f*y[i]", "float *z, const float *x, const float *y", [torch.float32] * 3),
      ("z[i] = x[i] - y[i] * z[i]", "double *z, const float *x, const float *y", [torch.float64] + [torch.float32] * 2),
      ("z[i] = x[i] + (float)y[i]", "bfloat16 *z, const half *x, const bfloat16 *y",
       [torch.bfloat16, torch.float16, torch.bfloat16]),
      ("z[i] = 0.5f * x[i] + (float)y[i]", "fp8_e4m3 *z, const bfloat16 *x, const fp8_e4m3 *y",
       [torch.float8_e4m3fn, torch.bfloat16, torch.float8_e4m3fn]),
      ("z[i] = x[i] * conj(y[i])", "complex64 *z, const complex64 *x, const complex64 *y", [torch.complex64] * 3),
      ("z[i] = x[i] + (i >= 2 ? y[i - 2] : 0) - (i + 1 < n ? y[i + 1] : 0)", "int *z, const int *x, const int *y",
       [torch.int32] * 3)]


@pytest.mark.parametrize("case", range(len(EW)))
@pytest.mark.parametrize("offsets", [(0, 0, 0), (0, 1, 0), (1, 0, 1), (0, 1, 2), (3, 2, 5)])
def test_elementwise_equals_one_element_kernel(dev, case, offsets):
    stmt, sig, dts = EW[case]
    k = hm.compile(stmt, sig, name="unal_ew")
    for n in SIZES:
        rng = np.random.default_rng(n + case)
        src = [values(dt, n + 16, rng).to(dev) for dt in dts]
        outs = []
        for cfg in (None, SCALAR):
            z = src[0].clone()
            views = [t[o:o + n] for t, o in zip([z, *src[1:]], offsets)]
            hm.elementwise(k, n, views, config=cfg)
            torch.cuda.synchronize()
            if cfg is None:
                assert tag(k) == "ew"
            outs.append(host_bits(z.view(torch.uint8)))
        assert np.array_equal(outs[0], outs[1]), (n, offsets)      # the elements around the view included


@pytest.mark.parametrize("offsets", [(0, 1), (1, 0), (2, 3)])
@pytest.mark.parametrize("fmt", ["int", "float", "bfloat16", "fp8_e4m3"])
def test_reductions(dev, fmt, offsets):
    """Products of small integers: every partial sum is exact in float and
    double, so each facility must return exactly the integer sum."""
    tdt = {"int": torch.int32, "float": torch.float32, "bfloat16": torch.bfloat16,
           "fp8_e4m3": torch.float8_e4m3fn}[fmt]
    h = hm.compile("x[i]*y[i]", f"float: const {fmt} *x, const {fmt} *y", name="unal_red")
    for n in SIZES:
        rng = np.random.default_rng(n)
        x, y = (rng.integers(-4, 5, n + 16) for _ in range(2))
        xd, yd = (torch.from_numpy(v.astype(np.float32)).to(tdt).to(dev)[o:o + n] for v, o in zip((x, y), offsets))
        p = x[offsets[0]:offsets[0] + n] * y[offsets[1]:offsets[1] + n]
        out = torch.empty((), device=dev)
        hm.reduce(h, None, "a+b", "0", n, [xd, yd], out)
        assert tag(h) == "rs1" and out.item() == p.sum()
        assert hm.reduce_compensated(h, n, [xd, yd]).item() == p.sum()
        if fmt != "fp8_e4m3" or n < 70001:
            want = np.sqrt(np.float64((p.astype(np.int64) ** 2).sum()))
            assert abs(hm.norm2(h, n, [xd, yd]).item() - want) <= 1e-6 * want
        sc = torch.empty(n, device=dev)
        hm.scan(h, "a+b", "0", n, [xd, yd], sc)
        assert np.array_equal(host_bits(sc).astype(np.int64), np.cumsum(p))
        off = np.array([0, n // 3, n // 3, n // 2 + 1 if n > 1 else 1, n])
        so = torch.empty(4, device=dev)
        hm.reduce_segmented(h, "a+b", "0", torch.from_numpy(off).to(dev), n, [xd, yd], so)
        assert so.tolist() == [p[a:b].sum() for a, b in zip(off, off[1:])]
