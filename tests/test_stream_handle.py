"""The stream handle that native calls get: torch's current stream, by the direct
function where torch has it and by the public interface where it has not."""
import types

import pytest
import torch

from paper_2410_08743_amd import render as R


def test_handle_without_the_direct_function(monkeypatch):
    monkeypatch.setattr(R, "_raw_stream", None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=0x1234))
    assert R._stream().value == 0x1234


@pytest.mark.gpu
@pytest.mark.parametrize("direct", [True, False])
def test_handle_is_the_current_streams(monkeypatch, direct):
    if not direct:
        monkeypatch.setattr(R, "_raw_stream", None)
    side = torch.cuda.Stream()
    assert side.cuda_stream != torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert R._stream().value == side.cuda_stream
    assert (R._stream().value or 0) == torch.cuda.current_stream().cuda_stream
