"""Calls in scratch memory of the caller give the results of calls in the library's
own, refuse too little of it, and run on streams other than the current one."""
import ctypes

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


def _p(t):
    return ctypes.c_void_p(t.data_ptr()) if t is not None else None


def _sigma(M, seed=3):
    import torch
    return torch.from_numpy(G.make_instance("m144_k5", M=M, seed=seed).sigma).to("cuda:0")


@pytest.mark.parametrize("M,K,flags,corr,mean", [(1, 1, 0, True, False), (9, 2, 1, False, False), (20, 4, 2, True, False),
                                                 (20, 4, 3, False, False), (17, 3, 16, True, False),
                                                 (17, 5, 1, True, True), (17, 5, 0, False, True)])
def test_forward(P, M, K, flags, corr, mean):
    import torch
    print("case: lent scratch, forward", M, K, flags, corr, mean, flush=True)
    L, s = P.lib(), _sigma(M)
    mu = torch.linspace(-0.4, 0.5, 2 * M, dtype=torch.float64, device="cuda:0") if mean else None
    n = P.gbs_total_outputs(M, K)
    out = [[torch.empty(n, dtype=torch.float64, device="cuda:0") if corr or q else None for q in range(2)] for _ in range(2)]
    if mean:
        st = L.gbs_cumulants_displaced(M, _p(s), _p(mu), K, flags, _p(out[0][0]), _p(out[0][1]), None)
    else:
        st = L.gbs_cumulants(M, _p(s), K, flags, _p(out[0][0]), _p(out[0][1]), None)
    assert st == P.GBS_OK
    need = L.gbs_cumulants_scratch(M, K, flags, mean, corr)
    work = torch.full((need,), 0xff, dtype=torch.uint8, device="cuda:0")  # whatever was there before
    torch.cuda.synchronize()
    args = (M, _p(s), _p(mu), K, flags, _p(out[1][0]), _p(out[1][1]), _p(work))
    assert L.gbs_cumulants_in(*args, need - 1, None) == P.GBS_E_OUT_OF_MEMORY
    assert L.gbs_cumulants_in(*args, need, None) == P.GBS_OK
    for a, b in zip(*out):
        assert a is None and b is None or torch.equal(a, b)


def test_other_calls(P):
    import torch
    print("case: lent scratch, adjoint, sampler, estimator, Pearson", flush=True)
    L, M, K = P.lib(), 14, 3
    s = _sigma(M)
    n = P.gbs_total_outputs(M, K)
    gen = torch.Generator(device="cuda:0").manual_seed(1)
    g = torch.randn(n, dtype=torch.float64, device="cuda:0", generator=gen)
    own = torch.empty_like(s)
    assert L.gbs_cumulant_grad(M, _p(s), K, 0, None, _p(g), _p(own), None) == P.GBS_OK
    assert torch.equal(P.gbs_cumulant_grad(M, s, K, grad_cum=g), own)
    assert L.gbs_cumulant_grad_in(M, _p(s), K, 0, None, _p(g), _p(own), _p(g), 8, None) == P.GBS_E_OUT_OF_MEMORY

    _, kap = P.gbs_cumulants(M, s, 5, P.GBS_PARITY)
    u = torch.rand((M, 100), dtype=torch.float64, device="cuda:0", generator=gen)
    bits, prob, _ = P.gbs_sample(M, kap, 5, u)
    b2, p2 = torch.empty_like(bits), torch.empty_like(prob)
    assert L.gbs_sample(M, _p(kap), 5, 100, _p(u), _p(b2), _p(p2), None, 0, 0, None) == P.GBS_OK
    assert torch.equal(bits, b2) and torch.equal(prob, p2)
    assert L.gbs_sample_in(M, _p(kap), 5, 100, _p(u), _p(b2), _p(p2), None, _p(g), 8, 0, None) == P.GBS_E_OUT_OF_MEMORY

    cum = P.gbs_sample_cumulants(bits, 3)
    c2 = torch.empty_like(cum)
    assert L.gbs_sample_cumulants(M, 100, _p(bits), 3, _p(c2), 0, None) == P.GBS_OK
    assert torch.equal(cum, c2)
    assert L.gbs_sample_cumulants_in(M, 100, _p(bits), 3, _p(c2), _p(g), 8, 0, None) == P.GBS_E_OUT_OF_MEMORY

    for m in (2, 16384, 16385, 300001):  # one workgroup up to 16,384
        x = torch.randn(m, dtype=torch.float64, device="cuda:0", generator=gen)
        y = x + torch.randn(m, dtype=torch.float64, device="cuda:0", generator=gen)
        r, r2 = P.gbs_pearson(x, y), torch.empty(1, dtype=torch.float64, device="cuda:0")
        assert L.gbs_pearson(m, _p(x), _p(y), _p(r2), 0, None) == P.GBS_OK
        assert torch.equal(r, r2)
        xc, yc = x - x.mean(), y - y.mean()
        ref = float((xc * yc).sum() / torch.sqrt((xc * xc).sum() * (yc * yc).sum()))
        assert abs(float(r) - ref) <= 1e-13


def test_other_stream(P):
    import torch
    print("case: lent scratch, other streams", flush=True)
    s = _sigma(24)
    ref = P.gbs_cumulants(24, s, 4)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    for stream in (side, side.cuda_stream, 0):
        got = P.gbs_cumulants(24, s, 4, stream=stream)
        torch.cuda.synchronize()
        assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])
