"""step_mf_apply with an event that was never recorded: such a torch event has
no handle, and the library must not be given none in its place (a prepare that
then waits for the event would run beside an apply that still reads its
workspace).  (CPU only: stand-ins for the event and the library.)"""
import pytest
import torch

from paper_2206_00470_amd import Store, store


class Event:
    def __init__(self, handle=0):
        self.cuda_event, self.records = handle, []

    def record(self, *stream):
        self.records.append(stream)
        self.cuda_event = self.cuda_event or 0x5000


class Lib:
    @staticmethod
    def ps_step_mf_apply(*args):
        Lib.event = args[-1].value
        return 0


@pytest.fixture
def handle(monkeypatch):
    monkeypatch.setattr(store, "lib", lambda: Lib)
    monkeypatch.setattr(store, "_stream", lambda s=None: None)
    s = Store.__new__(Store)
    s._loss = lambda loss: loss

    def given(**kw):
        s._h = None
        s.step_mf_apply(4, 0.1, torch.empty(8, dtype=torch.uint8), loss=torch.empty(1, dtype=torch.float64), **kw)
        return Lib.event
    return given


def test_an_event_gets_its_handle_before_the_call(handle):
    ev = Event()
    assert handle(rows_done=ev) == 0x5000 and ev.records == [()]
    side = object()
    ev = Event()
    assert handle(rows_done=ev, stream=side) == 0x5000 and ev.records == [(side,)]


def test_a_recorded_event_is_passed_as_it_is(handle):
    ev = Event(0x77)
    assert handle(rows_done=ev) == 0x77 and ev.records == []
    assert not handle()
