"""Step-by-step double elision (12 modes and more) against the sampler oracle:
odd and even mode counts (the last two-step pass ends on either side), one
sample, and ragged sample blocks; batches are bitwise equal to the whole call.  Tolerances are those of tests/test_gpu_sampler.py: the
conditionals carry the rounding of sums of at most C(M, 4) terms of order one."""
import numpy as np
import pytest

import gbs_inputs as G
import oracle as O
from test_gpu_sampler import P, _compare, _gpu_sample, _say  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,n", [(11, 65), (12, 1), (13, 64), (17, 65), (24, 130), (40, 1500), (41, 3000)])
def test_against_oracle(P, M, n):  # noqa: F811
    _say("case: double elision by steps", M, n)
    inst = G.make_instance("m144_k5", M=M, seed=900 + M)
    _, cum = O.c_forward(inst.sigma, 5, O.PARITY)
    u = G.sampler_uniforms(M, n, 901 + M)
    bits, prob, cond = _gpu_sample(P, cum, M, 5, u)
    assert _compare(cum, M, 5, u, bits, prob, cond, f"M={M}") <= 1


def test_batches_give_the_same_samples(P):  # noqa: F811
    M, n = 21, 400
    _say("case: double elision in batches", M, n)
    inst = G.make_instance("m144_k5", M=M, seed=77)
    _, cum = O.c_forward(inst.sigma, 5, O.PARITY)
    u = G.sampler_uniforms(M, n, 78)
    whole = _gpu_sample(P, cum, M, 5, u)
    for batch in (64, 200, 1000):
        part = _gpu_sample(P, cum, M, 5, u, batch)
        assert np.array_equal(whole[0], part[0])
        assert np.array_equal(whole[1], part[1])
        assert np.array_equal(whole[2], part[2])
