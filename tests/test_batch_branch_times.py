"""The rough step times by which a batch's groups are dealt to the branches of
its graph, called through the library's C++ symbols (CPU only)."""
import ctypes

import pytest

from paper_2308_02329_amd import _lib as L


def _dense(n, xs, js, slab):
    fn = L.load()._ZN4chym13dense_step_usEiiib
    fn.argtypes, fn.restype = [ctypes.c_int] * 3 + [ctypes.c_bool], ctypes.c_double
    return fn(n, xs, js, slab)


def _sparse(n, lrb):
    fn = L.load()._ZN4chym14sparse_step_usEii
    fn.argtypes, fn.restype = [ctypes.c_int] * 2, ctypes.c_double
    return fn(n, lrb)


@pytest.mark.parametrize("n,xs,slab,us", [(200, 1, False, 0.63), (200, 1, True, 1.44), (800, 1, False, 6.2), (800, 1, True, 14.0),
                                          (600, 3, False, 6.2)])
def test_dense_steps_as_measured(n, xs, slab, us):
    """Team (N = 200), slab and packed streamed-J kernels within 40%."""
    assert abs(_dense(n, xs, 1, slab) / us - 1.0) <= 0.4


def test_sparse_steps_go_with_the_blocks_units():
    assert abs(_sparse(800, 2) / 0.93 - 1.0) <= 0.4
    assert abs(_sparse(200, 1) / 0.23 - 1.0) <= 0.4
    assert _sparse(800, 0) < 0.5 * _sparse(800, 2)
