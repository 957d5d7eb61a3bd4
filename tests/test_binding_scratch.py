"""Which streams are lent memory of torch's allocator to work in: the default stream
and torch's own, never a handle that can stand for another queue later (the
allocator hands a block out again by the handle alone).  torch's CUDA functions are
replaced by recorders, so no GPU is needed."""
import contextlib

import pytest
import torch

from paper_2511_14923_amd import _binding as B

DEV = torch.device("cuda", 0)


class Stream:
    def __init__(self, handle, stream_id):
        self.cuda_stream, self.stream_id = handle, stream_id


def external(handle, device=None):  # torch's id of a stream that it did not make
    return Stream(handle, handle)


@pytest.fixture
def cuda(monkeypatch):
    """torch.cuda with a settable current stream; `lent` holds what was allocated and where."""
    class State:
        current = Stream(0, 0)
        capturing = False
        lent = []

    st = State()
    st.lent = []

    @contextlib.contextmanager
    def on(stream):
        old, st.current = st.current, stream
        yield
        st.current = old

    def empty(n, **kw):
        st.lent.append((n, st.current.cuda_stream))
        return n

    monkeypatch.setattr(torch.cuda, "Stream", Stream)
    monkeypatch.setattr(torch.cuda, "ExternalStream", external)
    monkeypatch.setattr(torch.cuda, "stream", on)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda d=None: st.current)
    monkeypatch.setattr(torch.cuda, "default_stream", lambda d=None: Stream(0, 0))
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: st.capturing)
    monkeypatch.setattr(torch, "empty", empty)
    return st


@pytest.mark.parametrize("handle", [1, 2, 0x7f0012345680])
def test_foreign_handles_get_none(cuda, handle):
    """2 is hipStreamPerThread: one handle, a queue in every thread."""
    assert B._scratch(4096, handle, DEV) is None
    assert B._scratch(4096, external(handle), DEV) is None
    cuda.current = external(handle)
    assert B._scratch(4096, None, DEV) is None
    assert cuda.lent == []


def test_torch_streams_are_lent_memory(cuda):
    pool = Stream(0x55d2c0de0000, 3)
    assert B._scratch(4096, pool, DEV) == 4096
    assert B._scratch(512, 0, DEV) == 512
    assert B._scratch(256, None, DEV) == 256
    cuda.current = pool
    assert B._scratch(128, None, DEV) == 128
    assert cuda.lent == [(4096, pool.cuda_stream), (512, 0), (256, 0), (128, pool.cuda_stream)]


def test_nothing_to_lend(cuda):
    assert B._scratch(0, None, DEV) is None
    assert B._scratch(-1, None, DEV) is None
    cuda.capturing = True
    assert B._scratch(4096, None, DEV) is None
    assert B._scratch(4096, Stream(8, 1), DEV) is None
    assert cuda.lent == []
