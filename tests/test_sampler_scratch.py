"""The scratch memory of a sampler call with a named batch, against the bounds that
the header states (no GPU needed: only an automatic batch asks for the free memory)."""
from math import comb

import pytest

import paper_2511_14923_amd as P


def _bytes(M, K, n, batch):
    return P.lib().gbs_sample_scratch(M, K, n, batch)


@pytest.mark.parametrize("M", [3, 20, 23, 24, 26, 144, 256])
@pytest.mark.parametrize("batch", [64, 128, 192, 4096, 65536])
def test_single_elision_takes_the_batch_as_named(M, batch):
    block = _bytes(M, 3, 64, 64)
    assert block <= 64 * 8 * (2 * comb(M + 1, 2) + 3 * M + 11)
    for n in (batch, 3 * batch):
        assert _bytes(M, 3, n, batch) == batch // 64 * block
    assert _bytes(M, 3, batch + 1, batch) == -(-(batch + 1) // 128) * block  # two equal parts


@pytest.mark.parametrize("M", [5, 11, 12, 40, 144, 200])
@pytest.mark.parametrize("batch", [64, 128, 4096])
def test_double_elision_keeps_to_the_memory_of_the_batch(M, batch):
    block = _bytes(M, 5, 64, 64)
    most = batch * 8 * (M + 4 + comb(M, 2) + comb(M + 1, 2) + comb(M, 3))
    for n in (batch, 10 * batch):
        assert 0 < _bytes(M, 5, n, batch) <= max(most, block)


def test_refused_arguments():
    assert _bytes(0, 3, 64, 64) == _bytes(257, 3, 64, 64) == _bytes(201, 5, 64, 64) == -1
    assert _bytes(20, 4, 64, 64) == _bytes(20, 3, -1, 64) == _bytes(20, 3, 64, -1) == -1
    assert _bytes(20, 3, 0, 64) == 0
