"""Which states the circuit simulation in LDS takes: those that fit what the device reports (64 KiB
without a device), the others go gate by gate."""
import ctypes as C

import pytest
import torch

from paper_2405_12866_amd import qfs as Q


@pytest.mark.skipif(torch.cuda.is_available(), reason="the rule of a device that reports more")
def test_states_beyond_the_lds():
    fits = Q.load()._ZN3qfs12circuit_fitsEi
    fits.argtypes, fits.restype = [C.c_int], C.c_bool
    # a state takes 2^n amplitudes of 16 bytes and a sixteenth more
    assert [n for n in range(16) if fits(n)] == [n for n in range(2, 14) if 17 << n <= 64 * 1024]
