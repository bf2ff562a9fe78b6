"""The workspace that the fused step allocates for itself: room for batch
records only where the device can spare it, and no allocation that fails first.
The device's memory is a stand-in here."""
import pytest
import torch

import paper_2404_09531_amd as om

GB = 1 << 30
SMALL, RECORDS = 1000, 8 * GB - 1000


class Device:
    """free, reserved and allocated bytes as torch reports them."""

    def __init__(self, mp, free, reserved=0, allocated=0, share=1.0, capturing=False):
        self.asked = []
        mp.setattr(torch.cuda, "is_current_stream_capturing", lambda: capturing)
        mp.setattr(torch.cuda, "mem_get_info", lambda device=None: (free, 288 * GB))
        mp.setattr(torch.cuda, "get_per_process_memory_fraction", lambda device=None: share)
        mp.setattr(torch.cuda, "memory_reserved", lambda device=None: reserved)
        mp.setattr(torch.cuda, "memory_allocated", lambda device=None: allocated)
        mp.setattr(om, "fwd_bwd_l2_records_size", lambda scene, n, n_max, delta, t_term: 0 if t_term else RECORDS)
        mp.setattr(om.torch, "empty", self.empty)

    def empty(self, shape, **kw):
        self.asked.append(shape[0])
        return None


class Handle:
    device = torch.device("cpu")


@pytest.mark.parametrize("what,kw,records", [
    ("an empty device", dict(free=250 * GB), True),
    ("four times the size", dict(free=32 * GB), True),
    ("less", dict(free=32 * GB - 1), False),
    ("the rest is cached", dict(free=24 * GB, reserved=20 * GB, allocated=12 * GB), True),
    ("cached, but maybe in pieces", dict(free=8 * GB - 1, reserved=100 * GB, allocated=0), False),
    ("in use", dict(free=24 * GB, reserved=20 * GB, allocated=13 * GB), False),
    ("a full device", dict(free=0), False),
    ("a share of the device", dict(free=250 * GB, share=0.1), False),
    ("a large share", dict(free=250 * GB, share=0.5, reserved=100 * GB, allocated=100 * GB), True),
    ("a share that is used up", dict(free=250 * GB, share=0.5, reserved=140 * GB), False),
    ("under capture", dict(free=250 * GB, capturing=True), False),
])
def test_records_only_where_there_is_room(monkeypatch, what, kw, records):
    dev = Device(monkeypatch, **kw)
    om._fwd_bwd_l2_workspace(Handle, 1 << 18, 256, om.DELTA, 0.0, SMALL)
    assert dev.asked == [SMALL + RECORDS if records else SMALL], what


def test_steps_without_records_do_not_ask(monkeypatch):
    dev = Device(monkeypatch, free=250 * GB)
    monkeypatch.setattr(torch.cuda, "mem_get_info", None)
    om._fwd_bwd_l2_workspace(Handle, 1 << 18, 256, om.DELTA, 1e-3, SMALL)
    om._fwd_bwd_l2_workspace(Handle, 0, 256, om.DELTA, 1e-3, 0)
    assert dev.asked == [SMALL, 1]
