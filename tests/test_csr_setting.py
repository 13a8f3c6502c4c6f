"""The reported tile setting of a CSR operator that was given none: the one its
FP64 products run with.  Host only."""
import ctypes

import pytest


@pytest.fixture(scope="module")
def L():
    import os
    from paper_1309_4616_amd import _binding
    if not os.path.exists(_binding.LIB_PATH):
        from paper_1309_4616_amd import build
        build.build()
    return _binding.lib()


def setting(L, n, new=None):
    op = ctypes.c_void_p()
    dummy = ctypes.c_void_p(1 << 20)
    assert L.expi_op_create_csr(ctypes.byref(op), n, 8 * n, dummy, dummy, dummy) == 0
    if new:
        assert L.expi_op_set_tiles(op, *new) == 0
    v, w, m = ctypes.c_int(), ctypes.c_int(), ctypes.c_int()
    assert L.expi_op_get_tiles(op, ctypes.byref(v), ctypes.byref(w), ctypes.byref(m)) == 0
    L.expi_op_destroy(op)
    return v.value, w.value, m.value


@pytest.mark.parametrize("n,want", [(2**15 - 1, (8, 4, 1)), (2**15, (4, 4, 1)), (98304, (4, 4, 1)), (98305, (8, 2, 1)),
                                    (2**17 - 1, (8, 2, 1)), (2**17, (8, 2, 1)), (2**17 + 1, (8, 2, 1)), (161468, (8, 2, 1)), (218453, (8, 2, 1)),
                                    (218454, (4, 4, 1)), (2**18, (4, 4, 1)), (2**18 + 1, (8, 2, 1)),
                                    (2**20, (4, 4, 1))])
def test_reported_setting_follows_the_rows(L, n, want):
    assert setting(L, n) == want


def test_given_setting_is_reported(L):
    assert setting(L, 2**16, (8, 4, 1)) == (8, 4, 1)
