"""Host side of the polynomial engine (CPU only), through the library's C++
functions: what they decide where no call reaches on its own."""
import ctypes
import os

import pytest

ifl = pytest.importorskip("paper_2404_07398_amd")

INF, NAN = float("inf"), float("nan")


def _function(name, restype, *argtypes):
    if not os.path.exists(ifl.LIB_PATH):
        pytest.skip("libifl.so not built")
    f = getattr(ifl.lib(), name)
    f.restype, f.argtypes = restype, argtypes
    return f


@pytest.mark.parametrize("res2,size2,bb,ok", [
    (1e-24, 1.0, 1.0, True), (1.1e-24, 1.0, 1.0, False),  # rtol = 1e-12
    (1e-24, 0.0, 0.0, False), (0.0, 0.0, 0.0, True),       # a zero field
    (7.8e-23, 1e8, 1.0, True), (7.9e-23, 1e8, 1.0, False),  # attainable: 8 u 1e4 = 8.9e-12
    (INF, INF, 1.0, False), (INF, 1.0, 1.0, False), (NAN, INF, 1.0, False),
    (1e-20, INF, 1.0, False), (1e-20, NAN, 1.0, False), (1e-25, INF, 1.0, True),
    (INF, INF, INF, True), (NAN, INF, INF, False),         # fields whose norm overflows
])
def test_columns_counted_as_converged(res2, size2, bb, ok):
    accepts = _function("_ZN3ifl12poly_acceptsEdddd", ctypes.c_bool, *[ctypes.c_double] * 4)
    assert accepts(res2, size2, bb, 1e-12) is ok
