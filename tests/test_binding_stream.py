"""The stream a call is put on: torch's current one, read through torch's raw
handle where this torch has it and through the public Stream object where not."""
from types import SimpleNamespace

import pytest
import torch

from paper_2412_06464_amd import gdn


def test_without_the_raw_handle(monkeypatch):
    asked = []

    def current(device):
        asked.append(device)
        return SimpleNamespace(cuda_stream=0x1234)

    monkeypatch.setattr(gdn, "_raw_stream", None)
    monkeypatch.setattr(torch.cuda, "current_stream", current)
    assert gdn._stream(torch.device("cuda", 0)) == 0x1234
    assert asked == [torch.device("cuda", 0)]


@pytest.mark.gpu
def test_both_ways_agree(monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    device = torch.device("cuda", 0)
    side = torch.cuda.Stream()
    for stream in (torch.cuda.current_stream(), side):
        with torch.cuda.stream(stream):
            fast = gdn._stream(device)
            with monkeypatch.context() as m:
                m.setattr(gdn, "_raw_stream", None)
                assert gdn._stream(device) == fast == stream.cuda_stream
