"""The step-by-step samplers against the sampler oracle:
odd and even mode counts (the last two-step pass ends on either side), one
sample, and ragged sample blocks; batches are bitwise equal to the whole call.  Tolerances are those of tests/test_gpu_sampler.py: the
conditionals carry the rounding of sums of at most C(M, 4) terms of order one."""
import numpy as np
import pytest

import gbs_inputs as G
import oracle as O
from test_gpu_sampler import P, _compare, _gpu_sample, _say  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,M,n", [(5, 11, 65), (5, 12, 1), (5, 13, 64), (5, 17, 65), (5, 24, 130), (5, 40, 1500),
                                   (5, 41, 3000), (3, 23, 65), (3, 24, 1), (3, 25, 64), (3, 33, 65),
                                   (3, 34, 129), (3, 101, 700), (3, 256, 70),
                                   (3, 25, 32768), (3, 26, 32769)])
def test_against_oracle(P, K, M, n):  # noqa: F811
    _say("case: sampler by steps", K, M, n)
    if M > 144:
        cum = G.synthetic_parity_cumulants(M, K, 7)
    else:
        inst = G.make_instance("m144_k5", M=M, seed=900 + M)
        _, cum = O.c_forward(inst.sigma, K, O.PARITY)
    u = G.sampler_uniforms(M, n, 901 + M)
    bits, prob, cond = _gpu_sample(P, cum, M, K, u)
    assert _compare(cum, M, K, u, bits, prob, cond, f"K={K} M={M}") <= 1


@pytest.mark.parametrize("K", [3, 5])
def test_batches_give_the_same_samples(P, K):  # noqa: F811
    M, n = 26, 400
    _say("case: batches", K, M, n)
    inst = G.make_instance("m144_k5", M=M, seed=77)
    _, cum = O.c_forward(inst.sigma, K, O.PARITY)
    u = G.sampler_uniforms(M, n, 78)
    whole = _gpu_sample(P, cum, M, K, u)
    for batch in (64, 200, 1000):
        part = _gpu_sample(P, cum, M, K, u, batch)
        assert np.array_equal(whole[0], part[0])
        assert np.array_equal(whole[1], part[1])
        assert np.array_equal(whole[2], part[2])
