"""Small reductions use the chip as larger ones do: one geometry, so that a map
that is slow per element (gathers, many arrays, divisions, a combine with
calls) is never left to a single block."""

import numpy as np
import pytest

from gpu_util import dev_array, need_gpu, torch
import paper_1304_5553_amd as hm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sig,expr,kinds", [
    ("float: const float *x, const int *k", "x[k[i]]", "fk"),
    ("float: " + ", ".join(f"const float *x{j}" for j in range(12)), " + ".join(f"x{j}[i]" for j in range(12)), "f" * 12),
    ("float: const int *a, const int *b", "(float)(a[i] % (b[i] + 3))", "kk")])
def test_the_kernel_of_a_large_call(sig, expr, kinds):
    dev = need_gpu()
    rng = np.random.default_rng(3)
    big = 70001
    arrays = [rng.integers(0, 4, big).astype(np.float32) if k == "f" else rng.integers(0, big, big).astype(np.int32)
              for k in kinds]
    h = hm.compile(expr, sig, name="smallred")
    xs = [dev_array(a) for a in arrays]
    seen = set()
    for n in (5000, 10922, 65536, big):
        out = torch.zeros((), device=dev)
        hm.reduce(h, None, "a+b", "0", n, xs, out)
        seen.update(h.last_symbols())
        a = [v[:n] for v in arrays]
        if kinds == "fk":
            want = arrays[0][a[1]].sum()
        elif kinds == "kk":
            want = float((a[0] % (a[1] + 3)).astype(np.float64).sum())
        else:
            want = float(sum(v.sum(dtype=np.float64) for v in a))
        assert abs(out.item() - want) <= 1e-6 * abs(want)
    assert len(seen) == 1
