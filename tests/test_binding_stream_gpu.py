"""The stream a call without one runs on: torch's current stream of the current device, inside and outside a stream context."""
import pytest

torch = pytest.importorskip("torch")

from paper_2602_11808_amd import binding

pytestmark = pytest.mark.gpu


def test_current_stream_is_torchs():
    side = torch.cuda.Stream()
    for _ in range(2):
        assert binding._stream(None) == int(torch.cuda.current_stream().cuda_stream)
        with torch.cuda.stream(side):
            assert binding._stream(None) == int(side.cuda_stream) == binding._stream(side)
        assert binding._current_stream_by_object() == binding._stream(None)
