"""The default stream of a call is torch's current stream: the raw handle the
binding passes equals the torch stream's own, on the default stream and inside
(nested) stream contexts."""
import pytest

from paper_2606_11718_amd import ccl
from tests.helpers import torch_mod

pytestmark = pytest.mark.gpu


def test_default_stream_is_torchs_current_stream():
    torch = torch_mod()
    torch.zeros(1, device="cuda")
    assert ccl._stream(None) == torch.cuda.current_stream().cuda_stream
    s, t = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(s):
        assert ccl._stream(None) == s.cuda_stream
        with torch.cuda.stream(t):
            assert ccl._stream(None) == t.cuda_stream
        assert ccl._stream(None) == s.cuda_stream
    assert ccl._stream(None) == torch.cuda.current_stream().cuda_stream
