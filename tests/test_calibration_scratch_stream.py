"""The calibrations' scratch memory comes from the pool of the stream that their kernels run on: the caching allocator may hand out
memory that earlier work of the current stream is still using, which is only safe in that stream's order.  (Shown on the CPU, with
the allocation and the library replaced; what a race does to the results is not a matter for a test.)"""
import types

import numpy as np
import pytest
import torch

from paper_2401_18079_amd import binding as B


class _Tensor:
    is_cuda, device = True, "cuda:0"

    def __init__(self, shape, dtype):
        self.shape, self.dtype = shape, dtype

    def dim(self):
        return len(self.shape)

    def is_contiguous(self):
        return True

    def numel(self):
        return int(np.prod(self.shape))

    def data_ptr(self):
        return 4096


@pytest.fixture
def allocations(monkeypatch):
    """Records (stream, bytes) of every device allocation while the library's calls do nothing."""
    seen, current = [], [None]

    class On:
        def __init__(self, stream):
            self.stream = stream

        def __enter__(self):
            self.before = current[0]
            if self.stream is not None:
                current[0] = self.stream

        def __exit__(self, *e):
            current[0] = self.before

    def empty(*shape, dtype=None, device=None, pin_memory=False):
        if device is not None:
            seen.append((current[0], shape[0]))
            return _Tensor(shape, dtype)
        return real(*shape, dtype=dtype)

    real = torch.empty
    lib = types.SimpleNamespace(kvq_calibrate_key_channels_workspace_bytes=lambda *a: 4096, kvq_calibrate_key_channels_ws=lambda *a: 0,
                                kvq_calibrate_workspace_bytes=lambda: 8192, kvq_calibrate_nuq=lambda *a: 0)
    monkeypatch.setattr(B, "load_library", lambda: lib)
    monkeypatch.setattr(B.torch, "empty", empty)
    monkeypatch.setattr(B.torch.cuda, "stream", On)
    monkeypatch.setattr(B.torch.cuda, "current_stream", lambda *a: types.SimpleNamespace(cuda_stream=0, synchronize=lambda: None))
    return seen


def _side_stream():
    return types.SimpleNamespace(cuda_stream=64, synchronize=lambda: None)


def test_key_channel_calibration(allocations):
    side = _side_stream()
    B.kvq_calibrate_key_channels(_Tensor((32768, 128), torch.float16), 0.01, stream=side)
    B.kvq_calibrate_key_channels(_Tensor((32768, 128), torch.float16), 0.01)
    assert allocations == [(side, 4096), (None, 4096)]


def test_signpost_calibration(allocations):
    side = _side_stream()
    x = _Tensor((1000,), torch.float32)
    B.kvq_calibrate_nuq(x, x, 2, 1, [-1, -0.3, 0.3, 1], stream=side)
    B.kvq_calibrate_nuq(x, x, 2, 1, [-1, -0.3, 0.3, 1])
    assert allocations == [(side, 8192), (None, 8192)]
