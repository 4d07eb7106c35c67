"""What the first call of an operation compiles: one program for all of its
kernels (a program costs about 0.1 s whatever it holds, and programs do not
compile side by side)."""

import pytest

from paper_1304_5553_amd import hipmr
import paper_1304_5553_amd as hm

torch = pytest.importorskip("torch")


def compiles():
    return hm.cache_stats()["compiles"]


def test_prepare_builds_one_program(tmp_path, monkeypatch):
    monkeypatch.setenv("HIPMR_CACHE_DIR", str(tmp_path))
    h = hm.compile("x[i]*(i % 3)", "float: const float *x", name="oneprog")
    before = compiles()
    assert hipmr.lib().hipmr_prepare_reduce(h.handle, b"a+b", b"0") == hipmr.OK
    assert compiles() == before + 1
    assert hipmr.lib().hipmr_prepare_reduce(h.handle, b"a+b", b"0") == hipmr.OK
    assert compiles() == before + 1
    assert hipmr.lib().hipmr_prepare_reduce(h.handle, b"max(a,b)", b"-INFINITY") == hipmr.OK
    assert compiles() == before + 2


@pytest.mark.gpu
def test_first_calls_build_one_program(tmp_path, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    monkeypatch.setenv("HIPMR_CACHE_DIR", str(tmp_path))
    n = 100003
    x = torch.ones(n, device="cuda")
    out, run = torch.zeros((), device="cuda"), torch.zeros(n, device="cuda")
    h = hm.compile("x[i]*(i % 5 + 1)", "float: const float *x", name="oneprog")
    for what in (lambda: hm.reduce(h, None, "a+b", "0", n, [x], out),
                 lambda: hm.scan(h, "a+b", "0", n, [x], run),
                 lambda: hm.reduce_compensated(h, n, [x]),
                 lambda: hm.norm2(h, n, [x], passes=1)):
        before = compiles()
        what()
        assert compiles() == before + 1
        what()
        assert compiles() == before + 1
    want = sum(k % 5 + 1 for k in range(n))
    assert out.item() == want and run[-1].item() == want


def test_the_cg_program_compiles_beside_torch(tmp_path, monkeypatch):
    """With the compiler that the process has once torch is loaded."""
    from paper_1304_5553_amd.cg import PoissonCG
    if torch.cuda.is_available():
        pytest.skip("covered by every CG test")
    monkeypatch.setenv("HIPMR_CACHE_DIR", str(tmp_path))
    before = compiles()
    with pytest.raises(hm.HipError):                 # compiled; nowhere to load it
        PoissonCG(8, 8, device="cpu", stream=0).solve(torch.zeros(64), 1)
    assert compiles() in (before, before + 1)        # before: by an earlier call in this process
