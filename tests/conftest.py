import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU and the built HIP library")


@pytest.fixture(scope="session")
def oracle():
    import oracle as _oracle
    _oracle._load()
    return _oracle


@pytest.fixture(scope="session")
def test_lib():
    """The library's test build, whose af1_test_* queries tell what its plans
    choose (plans are the same in both builds)."""
    import ctypes

    from paper_2609_06161_amd import build_lib
    L = ctypes.CDLL(build_lib.TEST_LIB)
    I = ctypes.c_int64
    L.af1_test_gemv_launches.argtypes = [I] * 4
    L.af1_test_multi_lds.argtypes = [I, I, I, ctypes.c_int32, I]
    L.af1_test_multi_lds.restype = I
    L.af1_test_gemm_form.argtypes = [I] * 4 + [ctypes.c_int32, ctypes.POINTER(ctypes.c_int32)]
    return L


@pytest.fixture(scope="session")
def gemm_form(test_lib):
    """gemm_form(m, n, r, T, product): (tile tokens, tile rows, K ranges, mixed
    grid) of one contraction; products 0 and 1 are the forward's, 2 and 3 the
    backward's."""
    import ctypes

    def form(m, n, r, T, product):
        f = (ctypes.c_int32 * 4)()
        assert test_lib.af1_test_gemm_form(m, n, r, T, product, f) == 0
        return tuple(f)
    return form
