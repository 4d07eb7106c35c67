"""The binding's marshalling extension (no GPU): it hands the C ABI function
the values the general path marshals, and leaves everything unusual alone."""

import ctypes

import numpy as np
import pytest
import torch

import paper_1304_5553_amd as hm
from paper_1304_5553_amd import hipmr as binding

VP = ctypes.c_void_p
EW = ctypes.CFUNCTYPE(ctypes.c_int32, VP, ctypes.c_int64, VP, VP, VP)
RED = ctypes.CFUNCTYPE(ctypes.c_int32, VP, ctypes.c_char_p, ctypes.c_char_p, ctypes.c_char_p, ctypes.c_int64,
                       VP, VP, VP, ctypes.c_size_t, VP, VP)


def slots(ptrs, count):
    array = ctypes.cast(ptrs, ctypes.POINTER(ctypes.POINTER(ctypes.c_uint64)))
    return [array[k][0] for k in range(count)]


@pytest.fixture(scope="module")
def fast():
    return binding._load_fast()


def test_values_equal_the_general_marshalling(fast):
    k = hm.compile("z[i] = a*x[i] + b*w[0] + (float)(c + d + e)",
                   "float *z, float a, const float *x, double b, const double *w, int c, unsigned d, long e")
    z, x, w = torch.zeros(8), torch.zeros(9), torch.zeros(1, dtype=torch.float64)
    seen = []

    def fn(h, n, ptrs, cfg, stream):
        seen.append((h, n, slots(ptrs, 8), cfg, stream))
        return 3
    cb = EW(fn)
    addr = ctypes.cast(cb, VP).value
    for scalars in ((0.1, -2.5, -1, 7, -(2 ** 40)), (1e300, float("inf"), 2 ** 31, 2 ** 32 - 1, 2 ** 63)):
        a, b, c, d, e = scalars
        args = [z, a, x, b, w, c, d, e]
        want = list(k.marshal(args)[0])
        st = fast.elementwise(addr, k._hv, k._kinds, args, 8, k._buffers()[2], 5)
        assert st == 3 and seen.pop() == (k._hv, 8, want, None, 5)
        assert fast.elementwise(addr, k._hv, k._kinds, tuple(args), 8, k._buffers()[2], 0) == 3
        assert seen.pop()[2] == want


def test_complex_scalars(fast):
    k = hm.compile("z[i] = a*z[i] + b", "complex64 *z, complex64 a, complex64 b")
    z = torch.zeros(8, dtype=torch.complex64)
    seen = []
    cb = EW(lambda h, n, ptrs, cfg, stream: seen.append(slots(ptrs, 3)) or 0)
    args = [z, 0.75 - 1.25j, complex(float("inf"), 1e300)]
    want = list(k.marshal(args)[0])
    assert fast.elementwise(ctypes.cast(cb, VP).value, k._hv, k._kinds, args, 8, k._buffers()[2], 0) == 0
    assert seen == [want]
    assert fast.elementwise(ctypes.cast(cb, VP).value, k._hv, k._kinds, [z, 1.0, 2j], 8, k._buffers()[2], 0) is None


def test_the_unusual_is_left_to_the_general_path(fast):
    k = hm.compile("z[i] = a*x[i]", "float *z, float a, const float *x")
    z, x = torch.zeros(8), torch.zeros(8)
    called = []
    cb = EW(lambda *a: called.append(a) or 0)
    addr = ctypes.cast(cb, VP).value
    param = torch.nn.Parameter(torch.zeros(8))
    sparse = torch.zeros(8).to_sparse()
    for args, n in (([z, 1.0, x], 9), ([z, 1.0], 8), ([z, 1, x], 8), ([z, np.float32(1), x], 8),
                    ([z, 1.0, param], 8), ([z, 1.0, x.data_ptr()], 8), ([z, 1.0, None], 8),
                    ([z, 1.0, sparse], 8), ([z, 1.0, x], np.int64(8)), ([z, 1.0, x], 2 ** 70),
                    (iter([z, 1.0, x]), 8)):
        assert fast.elementwise(addr, k._hv, k._kinds, args, n, k._buffers()[2], 0) is None
    for dtype in ("bfloat16", "half", "fp8_e4m3", "char"):
        kk = hm.compile("z[i] = x[i]", f"float *z, {dtype} a, const float *x")
        assert fast.elementwise(addr, kk._hv, kk._kinds, [z, 1.0, x], 8, kk._buffers()[2], 0) is None
        assert not kk._ordinary
    assert not called
    # outputs: dtype, length, layout, type
    f32 = torch.float32
    assert fast.out_pointer(z, f32, 8) == z.data_ptr()
    for out, dt, count in ((z, torch.int32, 8), (z, f32, 9), (torch.zeros(8, 2)[:, 0], f32, 8), (param, f32, 1),
                           (7, f32, 1), (z, None, 1), (z, f32, 2 ** 70)):
        assert fast.out_pointer(out, dt, count) is None


def test_reduce_passes_everything_through(fast):
    k = hm.compile("x[i]", "float: const float *x")
    x, ws = torch.zeros(8), torch.zeros(100, dtype=torch.int16)
    seen = []

    def fn(h, m, c, e, n, ptrs, out, w, wb, cfg, stream):
        seen.append((h, m, c, e, n, slots(ptrs, 1), out, w, wb, cfg, stream))
        return 0
    cb = RED(fn)
    addr = ctypes.cast(cb, VP).value
    for m in (None, b"x[i]"):
        assert fast.reduce(addr, k._hv, k._kinds, [x], 8, k._buffers()[2], 9, m, b"a+b", b"0", 4096, ws) == 0
        assert seen.pop() == (k._hv, m, b"a+b", b"0", 8, [x.data_ptr()], 4096, ws.data_ptr(), 200, None, 9)
    assert fast.reduce(addr, k._hv, k._kinds, [x], 8, k._buffers()[2], 9, None, "a+b", b"0", 4096, ws) is None
    assert fast.reduce(addr, k._hv, k._kinds, [x], 8, k._buffers()[2], 9, None, b"a+b", b"0", None, ws) is None
