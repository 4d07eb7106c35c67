"""The binding's cached workspaces (host side; no GPU)."""

import threading

import pytest

torch = pytest.importorskip("torch")

from paper_1304_5553_amd import hipmr  # noqa: E402


def test_each_thread_has_its_own():
    """Two threads that launch on one stream at a time must not share one."""
    got, both = {}, threading.Barrier(2)

    def take(k):
        both.wait()
        got[k] = [hipmr.workspace(1000, "cpu", 0x51) for _ in range(2)]
        both.wait()                                  # both alive until both have theirs
    threads = [threading.Thread(target=take, args=(k,)) for k in range(2)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    assert got[0][0] is got[0][1] and got[1][0] is got[1][1]
    assert got[0][0].data_ptr() != got[1][0].data_ptr()


def test_ended_threads_leave_theirs_to_the_next():
    before = len(hipmr._ws_cache)
    for _ in range(20):
        t = threading.Thread(target=hipmr.workspace, args=(1000, "cpu", 0x52))
        t.start()
        t.join()
    assert len(hipmr._ws_cache) == before + 1


def test_every_form_of_a_device():
    """A string, a torch.device, or whatever else torch takes (an index), as
    before: one buffer for the forms that read alike."""
    class Named:                                     # any object that torch.empty would take
        def __str__(self):
            return "cpu"
    a = hipmr.workspace(100, "cpu", 0x53)
    assert hipmr.workspace(100, torch.device("cpu"), 0x53) is a
    assert hipmr.workspace(100, Named(), 0x53) is a


def test_a_workspace_taken_over_has_one_owner():
    """However the ended thread named the device."""
    t = threading.Thread(target=hipmr.workspace, args=(1000, torch.device("cpu"), 0x54))
    t.start()
    t.join()
    buf = hipmr.workspace(1000, torch.device("cpu"), 0x54)
    owners = {k[2] for k, v in hipmr._ws_cache.items() if v is buf}
    assert owners == {threading.get_ident()}


def test_taking_over_leaves_other_devices_alone():
    """Streams of two devices may have the same number (0)."""
    t = threading.Thread(target=lambda: (hipmr.workspace(1000, "cpu", 0x55), hipmr.workspace(1000, "meta", 0x55)))
    t.start()
    t.join()
    ident = t.ident
    other = hipmr._ws_cache[("meta", 0x55, ident)]
    if threading.get_ident() != ident:
        hipmr.workspace(1000, "cpu", 0x55)
        assert hipmr._ws_cache[("meta", 0x55, ident)] is other
