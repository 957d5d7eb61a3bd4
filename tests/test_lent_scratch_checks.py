"""Lent scratch memory is checked on the host before anything is launched or read:
the pointers here are never dereferenced (no GPU needed)."""
import ctypes

import pytest

import paper_2511_14923_amd as P

BASE, HUGE = 0x10000, 1 << 50


def _calls(scratch, size):
    L, p = P.lib(), ctypes.c_void_p(0x1000)
    w = ctypes.c_void_p(scratch) if scratch else None
    yield L.gbs_cumulants_in(6, p, None, 3, 0, p, p, w, size, None)
    yield L.gbs_cumulants_in(6, p, p, 3, 0, None, p, w, size, None)
    yield L.gbs_cumulant_grad_in(6, p, 3, 0, p, p, p, w, size, None)
    yield L.gbs_sample_in(6, p, 3, 10, p, p, p, p, w, size, 0, None)
    yield L.gbs_sample_in(30, p, 5, 10, p, p, p, p, w, size, 0, None)
    yield L.gbs_sample_cumulants_in(6, 100, p, 3, p, w, size, 0, None)
    yield L.gbs_pearson_in(100000, p, p, p, w, size, 0, None)


@pytest.mark.parametrize("offset", [1, 8, 16, 64, 128, 255])
def test_misaligned_scratch_is_refused(offset):
    assert set(_calls(BASE + offset, HUGE)) == {P.GBS_E_INVALID_ARG}


def test_no_scratch_is_refused():
    assert set(_calls(0, HUGE)) == {P.GBS_E_INVALID_ARG}
    L, p = P.lib(), ctypes.c_void_p(0x1000)
    assert L.gbs_sample_in(6, p, 3, 0, p, p, p, p, None, 0, 0, None) == P.GBS_OK  # nothing to do


def test_negative_size_is_refused():
    assert set(_calls(BASE, -1)) <= {P.GBS_E_INVALID_ARG, P.GBS_E_OUT_OF_MEMORY}
