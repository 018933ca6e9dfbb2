"""GPU test: calls without a stream run on torch's current stream."""
import pytest
import torch

pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2606_02964_amd as msa


def test_current_stream_is_torchs():
    torch.zeros(1, device="cuda")
    side = torch.cuda.Stream()
    assert msa._stream(None) == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert msa._stream(None) == side.cuda_stream == torch.cuda.current_stream().cuda_stream
    assert msa._stream(None) == torch.cuda.current_stream().cuda_stream
    assert msa._stream(side) == side.cuda_stream and msa._stream(7) == 7
