"""Which subset a failed call names, where orders 1 and 2 are one launch: a mode that
is bad by itself comes before any pair, wherever the two lie in the launch."""
import numpy as np
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


def _bad(M, mode, pairs):
    """Vacuum with one bad mode and pairs of good modes with an indefinite block."""
    s = G.vacuum_covariance(M)
    if mode is not None:
        s[mode, mode] = s[mode + M, mode + M] = -0.9
    for a, b in pairs:
        for q in (0, M):
            s[a + q, b + q] = s[b + q, a + q] = 1.5  # Q = [[1, 1.5], [1.5, 1]]
    return s


def _calls(P, M, sigma):
    import torch
    s = torch.from_numpy(np.ascontiguousarray(sigma)).to("cuda:0")
    for K in (2, 3):
        g = torch.zeros(P.gbs_total_outputs(M, K), dtype=torch.float64, device="cuda:0")
        for call in (lambda: P.gbs_cumulants(M, s, K), lambda: P.gbs_cumulants(M, s, K, P.GBS_PARITY),
                     lambda: P.gbs_cumulant_grad(M, s, K, grad_cum=g)):
            with pytest.raises(P.GBSError) as e:
                call()
            assert e.value.status == P.GBS_E_NOT_SPD
            yield P.gbs_last_error()[1:]


@pytest.mark.parametrize("M,mode,pairs", [(300, 299, [(0, 1)]), (300, 70, [(0, 1), (2, 3), (298, 299)]),
                                          (20, 19, [(0, 1), (5, 9)])])
def test_a_bad_mode_comes_first(P, M, mode, pairs):
    print("case: bad mode and bad pairs", M, mode, pairs, flush=True)
    for _ in range(3):
        for order, rank in _calls(P, M, _bad(M, mode, pairs)):
            assert (order, rank) == (1, mode)


def test_a_bad_pair_alone(P):
    print("case: bad pair", flush=True)
    for order, rank in _calls(P, 40, _bad(40, None, [(3, 17)])):
        assert order == 2 and list(P.gbs_colex_unrank(order, rank)) == [3, 17]
