"""The adjoint's sums at the sizes where their loops end: one wavefront per
superset sum and one workgroup per mode pair (remainders around 64 and 256
terms), the smallest M of each order, each order's template, both conventions,
against the C oracle's reverse mode (1e-10 normwise, the tolerance of
tests/test_gpu_adjoint.py) and central differences."""
import math

import numpy as np
import pytest

import gbs_inputs as G
import oracle as O
from test_gpu_adjoint import P, _grad, _normwise, _say  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K", [(3, 3), (4, 4), (5, 5), (9, 5), (64, 2), (65, 3), (66, 3), (67, 2), (23, 4)])
def test_loss_gradient_matches_oracle(P, M, K):  # noqa: F811
    _say("case: adjoint pairs", M, K)
    inst = G.make_instance("grad_m144_k3", M=M, seed=500 + M)
    other = G.make_instance("grad_m144_k3", M=M, seed=900 + M)
    _, target = O.c_forward(other.sigma, K)
    _, kap = O.c_forward(inst.sigma, K)
    _, ref = O.c_loss_grad(inst.sigma, K, target)
    got = _grad(P, inst.sigma, K, gcum=2.0 * (kap - target))
    assert _normwise(got, ref) < 1e-10
    assert np.array_equal(got, got.T)


@pytest.mark.parametrize("M,K,conv", [(1, 1, 0), (5, 1, 0), (2, 2, 1), (7, 5, 1), (8, 5, 0)])
def test_both_gradients_against_differences(P, M, K, conv):  # noqa: F811
    _say("case: adjoint differences", M, K, conv)
    inst = G.make_instance("grad_m144_k3", M=M, seed=40 + M)
    N = O.total_outputs(M, K)
    rng = np.random.default_rng(M + 10 * K + conv)
    gc, gk = rng.standard_normal(N), rng.standard_normal(N)
    got = _grad(P, inst.sigma, K, gcorr=gc, gcum=gk, flags=conv)

    def f(s):
        c, k = O.correlators_and_cumulants(s, K, conv)
        return math.fsum(gc * c) + math.fsum(gk * k)

    h = 1e-6
    D = rng.standard_normal(inst.sigma.shape)
    D = 0.5 * (D + D.T)
    fd = (f(inst.sigma + h * D) - f(inst.sigma - h * D)) / (2 * h)
    # truncation h^2 and rounding u / h, as for the 1e-6 relative agreement of the
    # difference tests beside the adjoint
    assert abs(float((got * D).sum()) - fd) <= 1e-6 * max(1.0, abs(fd), float(np.abs(got * D).sum()))
