"""Calls whose launches would have 2^32 threads or more are refused before anything is
launched: the runtime would start what is left after the wrap, without an error.  (No GPU;
no pointer is dereferenced.)"""
import ctypes

import pytest

from test_abi_cpu import lib  # noqa: F401  (the module's fixture)

VP, I64, CI, SZ, CF = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int, ctypes.c_size_t, ctypes.c_float
FAKE, HUGE = 0x1000, 1 << 62


@pytest.mark.parametrize("C,K,n", [(1 << 22, 4096, 1000),      # k_search: a workgroup of 1024 threads per tile
                                   (1 << 26, 9, 1)])            # 64 threads per tile
def test_search(lib, C, K, n):  # noqa: F811
    for name in ("pwlq_search", "pwlq_search_fast"):
        f = getattr(lib, name)
        f.restype, f.argtypes = CI, [VP, I64, I64, CI, CI, CI, VP, VP, VP, VP, VP, SZ, VP]
        if name == "pwlq_search_fast" and K > 9:
            continue                                            # look-ups: launches of at most 2^21 tiles
        assert f(FAKE, C, K, 4, n, 0, FAKE, FAKE, FAKE, FAKE, FAKE, HUGE, None) == 1
        assert b"too large" in ctypes.cast(lib.pwlq_last_error, ctypes.CFUNCTYPE(ctypes.c_char_p))()


def test_quantize(lib):  # noqa: F811
    C, K = 1 << 23, 4096                                        # 2^35 elements, 2048 to a workgroup of 256
    lib.pwlq_quantize.restype, lib.pwlq_quantize.argtypes = CI, [VP, I64, I64, CI, CI, VP, VP, VP, VP, VP, VP]
    assert lib.pwlq_quantize(FAKE, C, K, 4, 0, FAKE, FAKE, FAKE, FAKE, FAKE, None) == 1
    lib.pwlq_quantize_packed.restype = CI
    lib.pwlq_quantize_packed.argtypes = [VP, I64, I64, CI, CI, VP, VP, VP, VP, VP, VP]
    assert lib.pwlq_quantize_packed(FAKE, C, K, 4, 0, FAKE, FAKE, FAKE, FAKE, FAKE, None) == 1


def test_selectors_and_error(lib):  # noqa: F811
    lib.pwlq_select_analytic.restype = lib.pwlq_mse.restype = CI
    lib.pwlq_select_analytic.argtypes = [VP, I64, I64, CI, CI, VP, VP, VP, SZ, VP]
    lib.pwlq_mse.argtypes = [VP, I64, I64, CI, CI, VP, VP, VP, VP, SZ, VP]
    assert lib.pwlq_select_analytic(FAKE, 1 << 26, 9, 0, 0, FAKE, FAKE, FAKE, HUGE, None) == 1
    assert lib.pwlq_mse(FAKE, 1 << 26, 9, 4, 0, FAKE, FAKE, FAKE, FAKE, HUGE, None) == 1


@pytest.mark.parametrize("M,N", [(8, 1 << 27), (63, 1 << 28), (64, 1 << 26)])
def test_inner_product(lib, M, N):  # noqa: F811
    lib.pwlq_linear_i8.restype = CI
    lib.pwlq_linear_i8.argtypes = [VP, I64, I64, CF, CF, VP, VP, I64, CI, VP, VP, VP, VP, VP, SZ, VP]
    assert lib.pwlq_linear_i8(FAKE, M, 16, 1.0, 0.0, FAKE, FAKE, N, 4, FAKE, FAKE, FAKE, None, FAKE, HUGE, None) == 1
