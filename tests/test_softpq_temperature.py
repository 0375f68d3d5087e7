"""The temperature's way to the host during the forward pass (softpq.py), with stand-ins for the device's side."""
import pytest
import torch

from paper_2302_03213_amd import softpq


class Device:
    """Records what is done while which device is the current one."""

    def __init__(self, monkeypatch, capturing=False):
        self.current, self.log, self.capturing = 0, [], capturing
        outer = self

        class Guard:
            def __init__(self, device):
                self.index = torch.device(device).index

            def __enter__(self):
                self.before, outer.current = outer.current, self.index

            def __exit__(self, *exc):
                outer.current = self.before

        class Event:
            def record(self):
                outer.log.append(("record", outer.current))

            def synchronize(self):
                outer.log.append(("synchronize", None))

        class Pinned:
            def copy_(self, source, non_blocking):
                outer.log.append(("copy", source.device.index))  # torch runs it on a stream of the source's device

            def __float__(self):
                return 2.5

        monkeypatch.setattr(torch.cuda, "device", Guard)
        monkeypatch.setattr(torch.cuda, "Event", Event)
        monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: self.capturing)
        monkeypatch.setattr(torch, "empty", lambda *args, **kwargs: Pinned())


class Temperature:
    is_cuda, shape, dtype = True, (), torch.float32

    def __init__(self, index):
        self.device = torch.device("cuda", index)

    def detach(self):
        return self


@pytest.mark.parametrize("index", [0, 1])
def test_event_follows_the_copy_on_the_temperatures_device(monkeypatch, index):
    device = Device(monkeypatch)
    host = softpq._HostTemperature(Temperature(index))
    assert device.log == [("copy", index), ("record", index)] and device.current == 0
    assert host.get() == 2.5 and device.log[-1][0] == "synchronize"


def test_a_capture_is_refused(monkeypatch):
    """A graph would keep the value that the temperature had when it was captured."""
    device = Device(monkeypatch)
    host = softpq._HostTemperature(Temperature(0))
    device.capturing = True
    with pytest.raises(RuntimeError, match="captured"):
        host.get()


def test_on_the_host_it_is_the_parameter_itself():
    temperature = torch.tensor(1.25)
    host = softpq._HostTemperature(temperature)
    assert host.event is None and host.get() == 1.25


def test_nothing_is_copied_where_no_backward_pass_can_follow():
    temperature = torch.tensor(1.25, requires_grad=True)
    assert softpq._host_temperature(None, None, temperature.detach(), None) is None
    with torch.no_grad():
        assert softpq._host_temperature(None, None, temperature, None) is None
    assert softpq._host_temperature(None, None, temperature, None).get() == 1.25
