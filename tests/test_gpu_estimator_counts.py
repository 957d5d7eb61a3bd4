"""The power sums behind the sample cumulants at the edges of their tiles (256
rows, 128 columns) and sample chunks (512), against plain FP64 arithmetic on the
host: counts are integers, so both sides differ by the rounding of the sum over
the partitions alone (at most 52 compensated terms of at most (d-1)! times the
largest moment product, 1: 1e-14 of it for the plain sum here)."""
import itertools
import math

import numpy as np
import pytest

from test_gpu_estimator import P  # noqa: F401

pytestmark = pytest.mark.gpu


def _partitions(items):
    if not items:
        yield []
        return
    head, rest = items[0], items[1:]
    for p in _partitions(rest):
        yield [[head]] + p
        for i in range(len(p)):
            yield p[:i] + [[head] + p[i]] + p[i + 1:]


def _reference(bits, K):
    """k-statistics of all subsets of orders 1..K, colex order, from integer counts."""
    n, M = bits.shape
    cols = [np.packbits(bits[:, k]) for k in range(M)]
    pop = np.array([bin(i).count("1") for i in range(256)])
    count = {}
    for d in range(1, K + 1):
        for S in itertools.combinations(range(M), d):
            v = cols[S[0]]
            for k in S[1:]:
                v = v & cols[k]
            count[S] = int(pop[v].sum())
    out = []
    for d in range(1, K + 1):
        terms = {}
        for pi in _partitions(list(range(d))):
            k = len(pi)
            w = (-1.0) ** (k - 1) * math.factorial(k - 1) / math.prod(n - i for i in range(k))
            for sg in _partitions(list(range(k))):
                v = w
                for g in sg:
                    v *= (-1.0) ** (len(g) - 1) * math.factorial(len(g) - 1)
                key = tuple(sorted(tuple(sorted(sum((pi[j] for j in g), []))) for g in sg))
                terms[key] = terms.get(key, 0.0) + v
        for S in sorted(itertools.combinations(range(M), d), key=lambda s: s[::-1]):
            out.append(math.fsum(c * math.prod(float(count[tuple(S[i] for i in b)]) for b in key)
                                 for key, c in terms.items()))
    return np.array(out)


@pytest.mark.parametrize("M,K,n", [(2, 2, 512), (2, 2, 511), (3, 3, 513), (24, 3, 1025), (25, 4, 700), (17, 5, 513),
                                   (140, 2, 2049), (5, 5, 40000)])
def test_counts_at_tile_edges(P, M, K, n):  # noqa: F811
    import torch
    print("case: power sums", M, K, n, flush=True)
    rng = np.random.default_rng(1000 * M + n)
    bits = (rng.random((n, M)) < rng.uniform(0.2, 0.95, M)).astype(np.uint8)
    got = P.gbs_sample_cumulants(torch.from_numpy(bits).to("cuda:0"), K).cpu().numpy()
    ref = _reference(bits, K)
    assert np.abs(got - ref).max() <= 52 * math.factorial(K - 1) * 1e-14


def test_unaligned_bits(P):  # noqa: F811
    import torch
    rng = np.random.default_rng(5)
    bits = (rng.random((300, 7)) < 0.5).astype(np.uint8)
    buf = torch.zeros(300 * 7 + 1, dtype=torch.uint8, device="cuda:0")
    buf[1:] = torch.from_numpy(bits).reshape(-1).to("cuda:0")
    got = P.gbs_sample_cumulants(buf[1:].view(300, 7), 3)
    assert torch.equal(got, P.gbs_sample_cumulants(torch.from_numpy(bits).to("cuda:0"), 3))


def test_counts_near_the_number_of_samples(P):  # noqa: F811
    """Every sample clicks in mode 0, all but one in mode 1: exact integer sums."""
    import torch
    n = (1 << 23) + 5
    print("case: large counts", n, flush=True)
    bits = torch.ones((n, 2), dtype=torch.uint8, device="cuda:0")
    bits[n // 3, 1] = 0
    got = P.gbs_sample_cumulants(bits, 2).cpu().numpy()
    assert got[0] == 1.0
    assert abs(got[1] - (n - 1) / n) <= 2.0 ** -53
    assert abs(got[2]) <= 1e-15  # mode 0 is constant: no covariance
