"""The stream that a call is given when it names none: the current stream's
handle, by torch's quick getters where both are there, else through
torch.cuda.current_stream().  No GPU needed."""
from types import SimpleNamespace

import pytest
import torch

from paper_2408_11052_amd import critic


@pytest.fixture
def torch_with_streams(monkeypatch):
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: SimpleNamespace(cuda_stream=11))
    return monkeypatch


def test_quick_getters(torch_with_streams):
    torch_with_streams.setattr(critic, "_raw_stream", lambda dev: 100 + dev)
    torch_with_streams.setattr(critic, "_device", lambda: 3)
    assert critic._stream() == 103


@pytest.mark.parametrize("missing", ["_raw_stream", "_device"])
def test_either_getter_missing(torch_with_streams, missing):
    torch_with_streams.setattr(critic, "_raw_stream", lambda dev: 100 + dev)
    torch_with_streams.setattr(critic, "_device", lambda: 3)
    torch_with_streams.setattr(critic, missing, None)
    assert critic._stream() == 11


def test_a_stream_that_is_named(torch_with_streams):
    assert critic._stream(SimpleNamespace(cuda_stream=7)) == 7


def test_a_device_that_is_not_initialised(torch_with_streams):
    torch_with_streams.setattr(torch.cuda, "is_initialized", lambda: False)
    assert critic._stream() == 11
