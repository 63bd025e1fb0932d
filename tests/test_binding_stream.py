"""The stream the binding passes on is torch's current one, also with a torch that has no short way to its handle."""
import pytest
import torch

from paper_2202_04305_amd import binding


@pytest.mark.parametrize("missing", ["_raw_stream", "_raw_device"])
def test_without_the_short_way(monkeypatch, missing):
    class Stream:
        cuda_stream = 0x1234

    monkeypatch.setattr(binding, missing, None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: Stream)
    assert binding._stream_ptr() == 0x1234


@pytest.mark.gpu
def test_both_ways_agree(monkeypatch):
    for stream in (torch.cuda.default_stream(), torch.cuda.Stream()):
        with torch.cuda.stream(stream):
            short = binding._stream_ptr()
            with monkeypatch.context() as m:
                m.setattr(binding, "_raw_stream", None)
                assert binding._stream_ptr() == short == stream.cuda_stream
