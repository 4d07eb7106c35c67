"""A solver on a stream of its own: dropped while its run is still going, and
captured before it has run, where another size has."""

import subprocess
import sys
import types

import pytest

from gpu_util import need_gpu, torch
from paper_1304_5553_amd.cg import PoissonCG

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("given", ["stream", "number", "object"])
def test_arrays_stay_until_the_run_ends(given):
    """The stream in each form the binding takes: torch's, its handle, or
    whatever holds that as cuda_stream."""
    dev = need_gpu()
    nx = 1024
    st = torch.cuda.Stream()
    b = torch.randn(nx * nx, device=dev)
    torch.cuda.synchronize()
    kept = PoissonCG(nx, nx, stream=st)
    want = kept.solve(b, 100)
    torch.cuda.synchronize()
    want = want.clone()
    for _ in range(5):
        on = {"stream": st, "number": st.cuda_stream, "object": types.SimpleNamespace(cuda_stream=st.cuda_stream)}[given]
        x = PoissonCG(nx, nx, stream=on).solve(b, 100)
        junk = [torch.full((nx * nx,), float("nan"), device=dev) for _ in range(12)]
        torch.cuda.synchronize()
        assert torch.equal(x, want)
        del junk, x


@pytest.mark.parametrize("first,then", [((32, 32), (1500, 1100)), ((1500, 1100), (32, 32))])
def test_capture_of_a_size_not_run_before(first, then):
    """The kernels of every size are loaded by the first run of any (in a
    process of its own: other tests run other sizes)."""
    need_gpu()
    code = f"""
import torch
from paper_1304_5553_amd.cg import PoissonCG
st = torch.cuda.Stream()
def rhs(nx, ny):
    return torch.ones(nx * ny, device="cuda")
PoissonCG(*{first}, stream=st).solve(rhs(*{first}), 4)
s = PoissonCG(*{then}, stream=st)
b = rhs(*{then})
torch.cuda.synchronize()
g = s.capture(6)
want = PoissonCG(*{then}, stream=st).solve(b, 12)
s.start(b)
for _ in range(2):
    g.launch(st)
torch.cuda.synchronize()
assert torch.equal(s.x, want)
print("done")
"""
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and r.stdout.strip().endswith("done"), r.stderr[-2000:]
