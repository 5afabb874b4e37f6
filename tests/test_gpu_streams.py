"""The raw calls run on the stream that is current on the current device, and on the one they are given."""
import numpy as np
import pytest
import torch

from paper_2104_05158_amd import tbe

pytestmark = pytest.mark.gpu


def test_calls_go_to_the_current_stream(gpu_device):
    side = torch.cuda.Stream()
    assert tbe._stream_ptr(None) == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert tbe._stream_ptr(None) == side.cuda_stream != torch.cuda.default_stream().cuda_stream
    assert tbe._stream_ptr(side) == side.cuda_stream

    lengths = torch.from_numpy(np.random.default_rng(1).integers(0, 9, 70_000).astype(np.int32)).to(gpu_device)
    want = np.concatenate([[0], np.cumsum(lengths.cpu().numpy(), dtype=np.int64)])
    scratch = torch.empty(tbe.tbe_inputs_scratch_bytes(70_000), dtype=torch.uint8, device=gpu_device)
    for inside in (True, False):
        out = torch.zeros(70_001, dtype=torch.int64, device=gpu_device)
        side.wait_stream(torch.cuda.current_stream())
        if inside:
            with torch.cuda.stream(side):
                assert tbe.tbe_lengths_to_offsets(lengths, 70_000, out, scratch) == tbe.TBE_OK
        else:
            assert tbe.tbe_lengths_to_offsets(lengths, 70_000, out, scratch, side) == tbe.TBE_OK
        side.synchronize()
        assert np.array_equal(out.cpu().numpy(), want)
