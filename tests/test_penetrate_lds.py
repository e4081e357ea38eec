"""LDS of the penetration test (no GPU): its launch counts on four blocks per CU, so for
every hand that a field can have four blocks' link segments fit the CU's 160 KB, and a
block holds at least one set per wave."""
import ctypes
import os

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_07418_amd", "liblg.so")


@pytest.mark.parametrize("F", range(1, 9))
def test_four_blocks_fit_a_compute_unit(F):
    if not os.path.exists(LIB):
        pytest.skip("no built library")
    lds = ctypes.CDLL(LIB)._ZN2lg17realize_lds_bytesEii
    lds.restype, lds.argtypes = ctypes.c_size_t, [ctypes.c_int, ctypes.c_int]
    for J in range(F, 8 * F + 1):
        sets, rest = divmod(lds(F, J) - 8 * J, 4 * 32 * J)  # four waves, 32 B per link of a set
        assert 4 * lds(F, J) <= 160 * 1024, (J, lds(F, J))
        assert 1 <= sets <= 64 // F and rest == 0, (J, sets, rest)
