"""The lists that Adam and the clears of several tensors take in one launch: what does not fit is
refused on the host, before any pointer is handed on."""
import pytest
import torch

from paper_2603_00145_amd import api


class _Lib:
    """Stands for the library: counts the launches."""
    def __init__(self):
        self.calls = 0

    def __getattr__(self, name):
        def call(*args):
            self.calls += 1
            return 0
        return call


@pytest.fixture
def lib(monkeypatch):
    lib = _Lib()
    monkeypatch.setattr(api, "load", lambda: lib)
    monkeypatch.setattr(api, "_stream", lambda: None)

    def need(t, dtype, name):       # host tensors stand for the device's
        if t.dtype != dtype or not t.is_contiguous():
            raise ValueError(name)
    monkeypatch.setattr(api, "_need", need)
    return lib


def _lists(sizes=(4, 6)):
    ts = [[torch.zeros(n) for n in sizes] for _ in range(4)]
    return ts + [[torch.zeros(sizes[0], dtype=torch.int16), None]]


def test_fitting_lists_are_taken(lib):
    api.adam_step_many(*_lists(), 1e-3, 1)
    assert lib.calls == 1


@pytest.mark.parametrize("which", range(1, 5))
def test_shorter_and_longer_lists_are_refused(lib, which):
    for change in (lambda ts: ts[:-1], lambda ts: ts + ts[:1]):
        ls = _lists()
        ls[which] = change(ls[which])
        with pytest.raises(ValueError):
            api.adam_step_many(*ls, 1e-3, 1)
    assert lib.calls == 0


@pytest.mark.parametrize("bad", [
    (1, torch.zeros(3)), (2, torch.zeros(5)), (3, torch.zeros(3)), (1, torch.zeros(4, device="meta")),
    (4, torch.zeros(3, dtype=torch.int16)), (4, torch.zeros(5, dtype=torch.int16)),
    (4, torch.zeros(4)), (4, torch.zeros(8, dtype=torch.int16)[::2]),
    (4, torch.zeros(4, dtype=torch.int16, device="meta"))])
def test_entries_that_do_not_fit_are_refused(lib, bad):
    ls = _lists()
    ls[bad[0]][0] = bad[1]
    with pytest.raises(ValueError):
        api.adam_step_many(*ls, 1e-3, 1)
    assert lib.calls == 0


class _DeviceTensor:
    """A device tensor as zero_many looks at it."""
    dtype, is_cuda = torch.float32, True

    def __init__(self, device):
        self.device_index, self.cleared = device, False

    def is_contiguous(self):
        return True

    def get_device(self):
        return self.device_index

    def data_ptr(self):
        return 0

    def numel(self):
        return 0

    def zero_(self):
        self.cleared = True


@pytest.mark.parametrize("devices,launches", [((0, 0), 1), ((0, 1), 0), ((1, 1), 0)])
def test_clears_go_to_the_current_device_only(lib, monkeypatch, devices, launches):
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    ts = [_DeviceTensor(d) for d in devices]
    api.zero_many(ts)
    assert lib.calls == launches
    assert all(t.cleared == (launches == 0) for t in ts)
