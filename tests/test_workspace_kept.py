"""The tensor given to set_workspace: kept while it is in use, and given up only behind what may still write to it.  No GPU: the
library's entry point and the device are stand-ins."""
import contextlib
import gc
import weakref

import pytest
import torch


class Buffer:
    is_cuda, device = True, 0

    def is_contiguous(self):
        return True

    def data_ptr(self):
        return 256

    def numel(self):
        return 4096

    def element_size(self):
        return 1

    def get_device(self):
        return 0


@pytest.fixture
def tcr(monkeypatch):
    from paper_1811_09736_amd import binding
    log = []

    class Library:
        status = binding.OK

        def tcr_set_workspace(self, pointer, size):
            log.append("set")
            return self.status

        def tcr_status_string(self, status):
            return b"refused"

    library = Library()
    monkeypatch.setattr(binding, "_lib", library)
    monkeypatch.setattr(binding, "_workspaces", {})
    monkeypatch.setattr(binding, "_replaced_in_capture", [])
    monkeypatch.setattr(torch.cuda, "device", lambda index: contextlib.nullcontext())
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: bool(getattr(library, "capturing", False)))
    monkeypatch.setattr(torch.cuda, "synchronize", lambda index: log.append(("finished", [r() is not None for r in log_refs])))
    log_refs = []
    return binding, library, log, log_refs


def given(tcr):
    binding, _, _, refs = tcr
    buffer = Buffer()
    refs.append(weakref.ref(buffer))
    binding.set_workspace(buffer)
    return refs[-1]


@pytest.mark.parametrize("successor", [True, False])
def test_the_device_has_finished_when_a_tensor_is_given_up(tcr, successor):
    binding, _, log, _ = tcr
    first = given(tcr)
    gc.collect()
    assert first() is not None and log == ["set"]
    second = given(tcr) if successor else binding.set_workspace(None)
    assert log == ["set", "set", ("finished", [True] * (2 if successor else 1))]      # (still there while the device finishes)
    gc.collect()
    assert first() is None
    assert second() is not None if successor else not binding._workspaces


def test_refused_or_given_again(tcr):
    binding, library, log, _ = tcr
    first = given(tcr)
    binding.set_workspace(first())
    library.status = binding.ERR_INVALID_ARG
    with pytest.raises(binding.TcrError):
        binding.set_workspace(Buffer())
    gc.collect()
    assert first() is not None and log == ["set"] * 3


def test_replaced_while_a_graph_is_recorded(tcr):
    binding, library, log, _ = tcr
    first = given(tcr)
    library.capturing = True
    binding.set_workspace(None)
    gc.collect()
    assert first() is not None and log == ["set", "set"]
