"""CPU checks of size limits that are refused on the host, before any device
work (the pointers are never read)."""
import ctypes as C

import pytest

from paper_1409_2065_amd import _lib


@pytest.mark.parametrize("n,k", [(12290, 12289), (16384, 12289), (16384, 16383)])
def test_knn_refuses_more_neighbours_than_it_can_rank(n, k):
    """A row's exact distances are ranked in the LDS of one block: 12288 at most."""
    lib = _lib.load()
    p, ne = C.c_void_p(16), C.c_int64(-1)
    st = lib.cc_build_knn_weights(n, 2, 0, p, 2, None, 2, k, 0.5, 0, p, p, p, n * k, C.byref(ne), None, None)
    assert st == _lib.CC_ERR_INVALID_ARG
    assert b"12288" in lib.cc_last_error_message()
    assert ne.value == -1
