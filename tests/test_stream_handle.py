"""The binding's stream handle is the current stream's, by either way of reading it."""
import pytest
import torch

from paper_1409_8186_amd import api


def test_without_the_raw_handle(monkeypatch):
    class Stream:
        cuda_stream = 77
    monkeypatch.setattr(api, "_raw_stream", None)
    monkeypatch.setattr(torch.cuda, "current_stream", Stream)
    assert api._stream() == 77


@pytest.mark.gpu
def test_both_ways_name_the_current_stream(monkeypatch):
    side = torch.cuda.Stream()
    for s in (torch.cuda.current_stream(), side):
        with torch.cuda.stream(s):
            raw = api._stream()
            with monkeypatch.context() as m:
                m.setattr(api, "_raw_stream", None)
                assert raw == api._stream() == s.cuda_stream
