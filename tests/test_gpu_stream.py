"""Calls go to the stream that is current for the current device, whichever way it is named."""
import pytest
import torch

import paper_2502_01776_amd as S

pytestmark = pytest.mark.gpu


def test_current_stream_handle():
    torch.zeros(1, device="cuda")
    side = torch.cuda.Stream()
    assert S.binding._stream(None) == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert S.binding._stream(None) == side.cuda_stream == torch.cuda.current_stream().cuda_stream
    assert S.binding._stream(None) == torch.cuda.current_stream().cuda_stream
    assert S.binding._stream(side) == S.binding._stream(side.cuda_stream) == side.cuda_stream
