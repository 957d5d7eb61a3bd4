"""Which orders a timed call reports: one entry per launch of the forward pass, in
the order of the launches, and none for an order without a launch of its own."""
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


@pytest.mark.parametrize("K,flags,orders", [(1, 0, [1]), (2, 0, [2]), (4, 1, [2, 3, 4]), (4, 2, [1, 2, 3, 4]),
                                            (3, 16, [1, 2, 3])])
def test_forward(P, K, flags, orders):
    import torch
    s = torch.from_numpy(G.make_instance("m144_k5", M=20, seed=3).sigma).to("cuda:0")
    print("case: timed orders", K, flags, flush=True)
    P.gbs_cumulants(20, s, K, flags | P.GBS_TIMING)
    t = P.gbs_last_timings()
    assert [o for st, o, _ in t if st == "forward"] == orders
    assert all(ms > 0.0 for _, _, ms in t)
    if not flags & P.GBS_MIXED:
        mu = torch.zeros(40, dtype=torch.float64, device="cuda:0")
        P.gbs_cumulants_displaced(20, s, mu, K, flags | P.GBS_TIMING)
        assert [o for st, o, _ in P.gbs_last_timings() if st == "forward"] == list(range(1, K + 1))


@pytest.mark.parametrize("K,orders", [(1, [1]), (3, [2, 3])])
def test_gradient(P, K, orders):
    import torch
    s = torch.from_numpy(G.make_instance("m144_k5", M=20, seed=3).sigma).to("cuda:0")
    g = torch.zeros(P.gbs_total_outputs(20, K), dtype=torch.float64, device="cuda:0")
    P.gbs_cumulant_grad(20, s, K, P.GBS_TIMING, grad_cum=g)
    assert [o for st, o, _ in P.gbs_last_timings() if st == "forward"] == orders
