"""A solver on a stream of its own, dropped while its run is still going."""

import pytest

from gpu_util import need_gpu, torch
from paper_1304_5553_amd.cg import PoissonCG

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("as_int", [False, True])
def test_arrays_stay_until_the_run_ends(as_int):
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
        x = PoissonCG(nx, nx, stream=st.cuda_stream if as_int else st).solve(b, 100)
        junk = [torch.full((nx * nx,), float("nan"), device=dev) for _ in range(12)]
        torch.cuda.synchronize()
        assert torch.equal(x, want)
        del junk, x
