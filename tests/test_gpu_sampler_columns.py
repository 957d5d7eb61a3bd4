"""A sample depends on its own column of uniforms alone: the same columns drawn in
calls of other sizes give the same bits, probabilities and conditionals, bit for
bit (one workgroup per 64 samples below 12 modes, or 24 with single elision; step
by step above)."""
import numpy as np
import pytest

import gbs_inputs as G
import oracle as O
from test_gpu_sampler import P, _gpu_sample, _say  # noqa: F401

pytestmark = pytest.mark.gpu


# with single elision 516 blocks of 64 samples are two groups of 258, 641 are 214, 214
# and 213, up to 383 are one group
@pytest.mark.parametrize("K,M,n", [(3, 10, 33000), (3, 26, 33000), (3, 26, 41000), (3, 57, 33000), (5, 9, 33000),
                                   (5, 14, 33000)])
def test_columns_do_not_depend_on_the_call(P, K, M, n):  # noqa: F811
    _say("case: columns", K, M, n)
    inst = G.make_instance("m144_k5", M=M, seed=60 + M)
    _, cum = O.c_forward(inst.sigma, K, O.PARITY)
    u = G.sampler_uniforms(M, n, 61 + M)
    bits, prob, cond = _gpu_sample(P, cum, M, K, u)
    for a, b in ((0, 1), (0, 400), (n - 300, n)):
        part = _gpu_sample(P, cum, M, K, u[:, a:b])
        assert np.array_equal(bits[a:b], part[0])
        assert np.array_equal(prob[a:b], part[1])
        assert np.array_equal(cond[:, a:b], part[2])
