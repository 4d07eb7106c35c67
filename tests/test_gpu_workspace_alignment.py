"""Workspaces at any address: the words that blocks exchange inside one launch
are 64 bits wide wherever the caller's buffer starts."""

import pytest

from gpu_util import host_bits, need_gpu, torch
import paper_1304_5553_amd as hm
from paper_1304_5553_amd.cg import PoissonCG

pytestmark = pytest.mark.gpu


def test_cg_refuses_a_misaligned_workspace():
    need_gpu()
    s = PoissonCG(64, 64)
    b = torch.ones(64 * 64, device="cuda")
    s._ws = torch.empty(s._ws.numel() + 8, dtype=torch.uint8, device="cuda")[4:]
    with pytest.raises(hm.WorkspaceError):
        s.start(b)


@pytest.mark.parametrize("shift", [1, 4, 7, 8])
@pytest.mark.parametrize("result,ctype,tdt", [("float", "float", torch.float32), ("long", "int", torch.int32)])
def test_any_workspace_address(shift, result, ctype, tdt):
    """The same bits as from an aligned workspace, and not a byte outside it."""
    dev = need_gpu()
    n = (1 << 23) + 5
    x = (torch.randint(-9, 9, (n,), dtype=tdt, device=dev) if tdt == torch.int32 else torch.randn(n, dtype=tdt, device=dev))
    h = hm.compile("x[i]", f"{result}: const {ctype} *x", name="wsalign")
    rdt = hm.torch_dtype(h.result_dtype)

    def within(nbytes, run):
        buf = torch.full((nbytes + 32,), 0xA5, dtype=torch.uint8, device=dev)
        got = run(buf[shift:shift + nbytes]).clone()
        edges = torch.cat([buf[:shift], buf[shift + nbytes:]])
        assert (edges == 0xA5).all()
        assert host_bits(got).tobytes() == host_bits(run(None)).tobytes()

    def reduce(ws):
        return hm.reduce(h, None, "a+b", "0", n, [x], torch.zeros((), dtype=rdt, device=dev), workspace_buf=ws)

    def scan(ws):
        return hm.scan(h, "a+b", "0", n, [x], torch.zeros(n, dtype=rdt, device=dev), workspace_buf=ws)
    within(hm.reduce_workspace_bytes(h, n), reduce)
    within(hm.scan_workspace_bytes(h, n), scan)
    if result == "float":
        for scale in (1.0, 2.0 ** 60):           # the norm's first pass stands, or its second is needed
            y = x * scale
            within(hm.reduce_workspace_bytes(h, n), lambda ws: hm.reduce_compensated(h, n, [y], workspace_buf=ws))
            for passes in (1, 2):
                within(hm.reduce_workspace_bytes(h, n),
                       lambda ws: hm.norm2(h, n, [y], passes=passes, workspace_buf=ws))
