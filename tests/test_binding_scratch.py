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
    monkeypatch.setattr(torch, "UntypedStorage", empty)
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


@pytest.fixture
def memory(cuda, monkeypatch):
    """Device memory of `total` bytes with `reserved` held by torch, `used` of it in use."""
    cuda.total, cuda.reserved, cuda.used, cuda.emptied = 288 << 30, 0, 0, 0

    def empty_cache():
        cuda.reserved, cuda.emptied = cuda.used, cuda.emptied + 1

    monkeypatch.setattr(torch.cuda, "mem_get_info", lambda d=None: (cuda.total - cuda.reserved, cuda.total))
    monkeypatch.setattr(torch.cuda, "memory_reserved", lambda d=None: cuda.reserved)
    monkeypatch.setattr(torch.cuda, "memory_allocated", lambda d=None: cuda.used)
    monkeypatch.setattr(torch.cuda, "empty_cache", empty_cache)
    return cuda


@pytest.mark.parametrize("stream", [None, 0, 2, Stream(8, 1)])
def test_out_of_memory_is_tried_again_without_torchs_unused_memory(memory, stream):
    need = 250 << 30

    def call():
        call.n += 1
        return B.GBS_OK if memory.total - memory.reserved >= need else B.GBS_E_OUT_OF_MEMORY

    call.n = 0
    memory.reserved, memory.used = 72 << 30, 1 << 30
    assert B._own(call, stream, DEV) == B.GBS_OK
    assert (call.n, memory.emptied) == (2, 1)
    # nothing unused, in use, or a stream under capture: the status stands
    call.n = 0
    memory.reserved = memory.used = 72 << 30
    assert B._own(call, stream, DEV) == B.GBS_E_OUT_OF_MEMORY
    memory.used, memory.capturing = 0, True
    assert B._own(call, stream, DEV) == B.GBS_E_OUT_OF_MEMORY
    assert (call.n, memory.emptied) == (2, 1)
    call.n = 0
    assert B._own(lambda: B.GBS_E_NOT_SPD, stream, DEV) == B.GBS_E_NOT_SPD


def test_automatic_batch_counts_torchs_unused_memory_as_free(memory, monkeypatch):
    per = 8_000_000  # bytes of tables per sample

    class Lib:
        @staticmethod
        def gbs_sample_scratch(M, K, n, batch):
            if n == 0 or batch < 0:
                return 0 if n == 0 else -1
            most = batch if batch else (memory.total - memory.reserved) // 4 // per
            most = min(max(64, most // 64 * 64), -(-n // 64) * 64)
            parts = -(-n // most)
            return per * (-(-(-(-n // parts)) // 64) * 64)

    monkeypatch.setattr(B, "lib", lambda: Lib)
    first = B._sample_bytes(144, 5, 16384, 0, DEV)
    assert first == per * 8192  # two equal parts
    memory.reserved = first     # as the first call leaves it
    assert Lib.gbs_sample_scratch(144, 5, 16384, 0) < first
    assert B._sample_bytes(144, 5, 16384, 0, DEV) == first
    memory.used = 60 << 30      # of it in use now: a quarter of what is left
    assert B._sample_bytes(144, 5, 16384, 0, DEV) == per * 5504
    assert B._sample_bytes(144, 5, 100, 0, DEV) == per * 128
    assert B._sample_bytes(144, 5, 16384, 640, DEV) == Lib.gbs_sample_scratch(144, 5, 16384, 640)
    assert B._sample_bytes(144, 5, 0, 0, DEV) == 0
    assert B._sample_bytes(144, 5, 10, -1, DEV) == -1


def test_lent_memory_is_not_filled(cuda, monkeypatch):
    """Deterministic algorithms have torch.empty fill what it returns, gigabytes here."""
    from torch.utils._python_dispatch import TorchDispatchMode

    class Seen(TorchDispatchMode):
        ops = []

        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            self.ops.append(str(func))
            return func(*args, **(kwargs or {}))

    monkeypatch.undo()
    monkeypatch.setattr(torch.cuda, "current_stream", lambda d=None: Stream(0, 0))
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: False)
    before = torch.are_deterministic_algorithms_enabled()
    torch.use_deterministic_algorithms(True)
    try:
        with Seen() as seen:
            work = B._scratch(4096, None, torch.device("cpu"))
    finally:
        torch.use_deterministic_algorithms(before)
    assert seen.ops == []
    assert work.nbytes() == 4096 and work.data_ptr()
