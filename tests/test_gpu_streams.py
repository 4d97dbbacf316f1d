"""The binding launches on torch's current stream of the current device."""

import pytest
import torch

from paper_2309_04671_amd import lib

pytestmark = pytest.mark.gpu


def test_stream_ptr_is_the_current_stream(gpu_lib):
    assert (lib.stream_ptr().value or 0) == torch.cuda.current_stream().cuda_stream
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        assert lib.stream_ptr().value == s.cuda_stream
        with torch.cuda.stream(torch.cuda.default_stream()):
            assert (lib.stream_ptr().value or 0) == torch.cuda.default_stream().cuda_stream
        assert lib.stream_ptr().value == s.cuda_stream
    assert lib.stream_ptr(s).value == s.cuda_stream
