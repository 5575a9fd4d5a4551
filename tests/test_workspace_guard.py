"""The binding's guard against one attention workspace in two calls at once, with the streams and events played on the CPU."""
import types

import pytest
import torch

from paper_2604_20503_amd import binding


class Event:
    made = []

    def __init__(self):
        self.on, self.done = None, False
        Event.made.append(self)

    def record(self, stream):
        self.on, self.done = stream, False

    def query(self):
        return self.done


@pytest.fixture
def at(monkeypatch):
    """Sets the current (device, stream handle)."""
    now = types.SimpleNamespace(place=(0, 0))
    monkeypatch.setattr(binding, "_ws_last_use", {})
    monkeypatch.setattr(binding, "_device_and_stream", lambda: now.place)
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: False)
    monkeypatch.setattr(torch.cuda, "Event", Event)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: now.place)
    monkeypatch.setattr(Event, "made", [])
    return lambda *place: setattr(now, "place", place)


def use(ws):
    binding._note_workspace_use(binding._guard_workspace(ws))


def test_default_streams_of_two_devices_are_two_streams(at):
    ws = torch.empty(16, dtype=torch.uint8)
    use(ws)
    use(ws)
    assert len(Event.made) == 1  # the second call follows the first on its stream
    at(1, 0)
    with pytest.raises(binding.FsrError):  # the first device's call may still run
        use(ws)
    Event.made[0].done = True
    use(ws)
    assert [e.on for e in Event.made] == [(0, 0), (1, 0)]  # watched where it was enqueued
    at(0, 0)
    with pytest.raises(binding.FsrError):
        use(ws)


def test_streams_of_one_device(at):
    ws = torch.empty(16, dtype=torch.uint8)
    at(0, 5)
    use(ws)
    at(0, 7)
    with pytest.raises(binding.FsrError):
        use(ws)
    use(torch.empty(16, dtype=torch.uint8))  # another workspace
    Event.made[0].done = True
    use(ws)
    assert Event.made[-1].on == (0, 7)
