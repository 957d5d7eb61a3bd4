"""Calls on several streams at once, from several threads, without waiting for each
other: torch's streams work in lent memory, a stream that torch did not make in the
library's own."""
import threading

import pytest

import gbs_inputs as G

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    import paper_2511_14923_amd as P
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    P.lib()
    return P


def test_streams_are_told_apart(P):
    import torch
    from paper_2511_14923_amd import _binding as B
    dev = torch.device("cuda", 0)
    side = torch.cuda.Stream()
    assert B._scratch(4096, side, dev) is not None
    assert B._scratch(4096, 0, dev) is not None
    assert B._scratch(4096, side.cuda_stream, dev) is None
    assert B._scratch(4096, torch.cuda.ExternalStream(side.cuda_stream), dev) is None
    with torch.cuda.stream(side):
        assert B._scratch(4096, None, dev) is not None
    with torch.cuda.stream(torch.cuda.ExternalStream(side.cuda_stream)):
        assert B._scratch(4096, None, dev) is None


@pytest.mark.parametrize("raw", [False, True])
def test_asynchronous_calls_of_two_threads(P, raw):
    import torch
    print("case: two threads, asynchronous", raw, flush=True)
    M, K = 40, 4
    sig = [torch.from_numpy(G.make_instance("m144_k5", M=M, seed=s).sigma).to("cuda:0") for s in (1, 2)]
    ref = [P.gbs_cumulants(M, s, K) for s in sig]
    streams = [torch.cuda.Stream() for _ in sig]
    n = P.gbs_total_outputs(M, K)
    out = [[torch.zeros((2, n), dtype=torch.float64, device="cuda:0") for _ in range(8)] for _ in sig]
    torch.cuda.synchronize()
    errors = []

    def work(i):
        try:
            for o in out[i]:
                P.gbs_cumulants(M, sig[i], K, P.GBS_ASYNC, corr=o[0], cum=o[1],
                                stream=streams[i].cuda_stream if raw else streams[i])
            streams[i].synchronize()
        except Exception as e:  # reported by the test's thread
            errors.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors
    for i in range(2):
        for o in out[i]:
            assert torch.equal(o[0], ref[i][0]) and torch.equal(o[1], ref[i][1])


def test_automatic_batch_after_other_calls(P, monkeypatch):
    """A memory-bound sampler call asks for the same scratch memory whether or not
    torch holds memory that an earlier call has used (a third of what is free; the
    sizes may differ by what the runtime itself takes meanwhile)."""
    import torch
    from paper_2511_14923_amd import _binding as B

    class Asked(Exception):
        pass

    def record(nbytes, *where):
        raise Asked(nbytes)

    M, n = 100, 1 << 17
    kap = torch.zeros(P.gbs_total_outputs(M, 5), dtype=torch.float64, device="cuda:0")
    u = torch.zeros((M, n), dtype=torch.float64, device="cuda:0")
    monkeypatch.setattr(B, "_scratch", record)
    asked = []
    torch.cuda.empty_cache()
    for hold in (0, torch.cuda.mem_get_info()[0] // 3):
        if hold:
            work = torch.empty(hold, dtype=torch.uint8, device="cuda:0")
            del work
        with pytest.raises(Asked) as e:
            P.gbs_sample(M, kap, 5, u, want_prob=False)
        asked.append(e.value.args[0])
    torch.cuda.empty_cache()
    whole = P.lib().gbs_sample_scratch(M, 5, 64, 64) * (n // 64)
    assert 0 < asked[0] < whole  # more than one part
    assert abs(asked[1] - asked[0]) <= 0.02 * asked[0]
