"""Host check (no GPU): the parts of the solve's workspace that the band reduction borrows
hold what it writes there, at every small order and at the orders where its tiles change."""
import ctypes
import os

import pytest

from paper_1904_05575_amd import _lib as L

ORDERS = list(range(1, 700)) + [1023, 1024, 1025, 2047, 2048, 2049, 2063, 2064, 2065, 4096, 4111,
                                4112, 4113, 6144, 10368, 32768]


def _desc(n):
    return L.BseDesc(nk=1, nv=1, nc=n, ng=9, coupling=L.BSE_TDA,
                     type=L.BSE_SINGLET, prec=L.BSE_PREC_FP64, split_terms=0, kappa=1.0,
                     scissor=0.0, ld=n)


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(L.LIB_PATH):
        pytest.fail("libbse.so is not built (run `python -m paper_1904_05575_amd.build`)")
    return L.lib()


def test_borrowed_parts_hold_the_reduction(lib):
    fits = getattr(lib, "_Z15solve_band_fitsPK8bse_desc")  # internal, C++ linkage
    fits.restype = ctypes.c_bool
    for n in ORDERS:
        assert fits(ctypes.byref(_desc(n))), n

