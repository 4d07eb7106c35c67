"""What the conjugate-gradient solver refuses before anything is launched (host
side; no GPU)."""

import pytest

torch = pytest.importorskip("torch")

import paper_1304_5553_amd as hm  # noqa: E402
from paper_1304_5553_amd.cg import PoissonCG  # noqa: E402


@pytest.mark.parametrize("b", [None, 0])
def test_no_right_hand_side(b):
    """Not a request to go on from the state there is."""
    s = PoissonCG(8, 8, device="cpu", stream=0)
    s.parity = 1
    with pytest.raises(hm.InvalidError):
        s.start(b)
    with pytest.raises(hm.InvalidError):
        s.solve(b, 0)
    assert s.parity == 1


def test_short_right_hand_side():
    with pytest.raises(hm.InvalidError):
        PoissonCG(8, 8, device="cpu", stream=0).start(torch.zeros(63))
