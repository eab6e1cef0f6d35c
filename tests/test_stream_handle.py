"""The stream handle of a call: the given stream's, else the current one's, with or without torch's
function for the bare handle."""

import pytest
import torch

from paper_2407_11349_amd import _lib


class _Stream:
    def __init__(self, handle):
        self.cuda_stream = handle


def test_a_given_stream_is_taken():
    assert _lib.stream_handle(_Stream(1234)) == 1234


def test_the_current_stream_without_the_bare_handle(monkeypatch):
    monkeypatch.setattr(_lib, "_raw_stream", None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: _Stream(77))
    assert _lib.stream_handle() == 77


def test_the_current_stream_by_the_bare_handle(monkeypatch):
    monkeypatch.setattr(_lib, "_raw_stream", lambda device: 500 + device)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    assert _lib.stream_handle() == 503


@pytest.mark.gpu
def test_both_ways_agree(monkeypatch):
    side = torch.cuda.Stream()
    for stream in (torch.cuda.default_stream(), side):
        with torch.cuda.stream(stream):
            bare = _lib.stream_handle()
            monkeypatch.setattr(_lib, "_raw_stream", None)
            assert _lib.stream_handle() == bare == int(stream.cuda_stream)
            monkeypatch.undo()
