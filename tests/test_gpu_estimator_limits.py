"""The sample cumulants at the ends of their range: the most samples that a call
takes (2^32 - 1, counts in 32 bits), packings in more than one row of a launch, and
the most modes."""
import numpy as np
import pytest

from test_gpu_estimator import P  # noqa: F401
from test_gpu_estimator_counts import _reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(1 << 32) - 1, (1 << 32) - 512, (1 << 28) + 257])
def test_most_samples(P, n):  # noqa: F811
    """One mode, two zeros: the mean is an exact quotient of integers."""
    import torch
    print("case: samples", n, flush=True)
    bits = torch.ones((n, 1), dtype=torch.uint8, device="cuda:0")
    bits[0, 0] = 0
    bits[n - 1, 0] = 0
    got = P.gbs_sample_cumulants(bits, 1).item()
    assert abs(got - (n - 2) / n) <= 2.0 ** -53


@pytest.mark.parametrize("M,K,n", [(256, 2, 600), (255, 2, 257), (256, 1, 3)])
def test_most_modes(P, M, K, n):  # noqa: F811
    import torch
    print("case: modes", M, K, n, flush=True)
    rng = np.random.default_rng(M + n)
    bits = (rng.random((n, M)) < rng.uniform(0.2, 0.95, M)).astype(np.uint8)
    got = P.gbs_sample_cumulants(torch.from_numpy(bits).to("cuda:0"), K).cpu().numpy()
    # counts are integers; at most two products of moments of at most 1 per subset
    assert np.abs(got - _reference(bits, K)).max() <= 1e-14
