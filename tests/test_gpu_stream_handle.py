"""The stream that the binding hands to the library is torch's current one, with and without the short way to it."""
import pytest
import torch

from paper_2206_01861_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("short_way", [True, False])
def test_stream_is_torchs_current_one(monkeypatch, short_way):
    if not short_way:
        monkeypatch.setattr(binding, "_raw_stream", None)
    assert binding._stream() == torch.cuda.current_stream().cuda_stream
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert binding._stream() == side.cuda_stream
    assert binding._stream() == torch.cuda.current_stream().cuda_stream
