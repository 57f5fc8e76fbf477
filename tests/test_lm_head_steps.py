"""The host's choice of vocabulary rows per backward step in the chunked LM head, which runs between
two launches of every such call (CPU only)."""
import ctypes as C
import time

import pytest

from paper_2605_12070_amd import _lib


def _step():
    # dppo::lmh_backward_step(T, d, V, chunk, dhidden, dweight)
    f = _lib.lib()["_ZN4dppo17lmh_backward_stepEllllbb"]
    f.restype, f.argtypes = C.c_int64, [C.c_int64] * 4 + [C.c_bool] * 2
    return f


# chunks of the 64 MiB scratch, and a caller's own over the longest vocabulary
@pytest.mark.parametrize("T,d,V,chunk", [(128, 512, 151936, 151808), (230, 2048, 151936, 141056),
                                         (256, 512, 151936, 126208), (300, 4096, 151936, 107008),
                                         (512, 2048, 151936, 60672), (2048, 4096, 151936, 11520),
                                         (64, 64, 1 << 21, 1 << 19), (65536, 4096, 151936, 2048),
                                         (16, 8, 5000, 256)])
def test_step_choice_is_quick_and_in_range(T, d, V, chunk):
    """Some tens of microseconds at any size (trying every multiple of 256 rows took 2 ms at
    T = 256), and a multiple of 256 rows between a quarter of the chunk and the chunk."""
    f = _step()
    best = min(_timed(f, T, d, V, chunk) for _ in range(5))
    assert best < 400e-6, best
    for dh in (True, False):
        for dw in (True, False):
            c = f(T, d, V, chunk, dh, dw)
            assert c % 256 == 0 and max(256, chunk // 4) <= c <= chunk


def _timed(f, *args):
    t0 = time.perf_counter()
    f(*args, True, True)
    return time.perf_counter() - t0


def test_step_choice_of_the_large_micro_batch():
    """T = 2048, d = 4096, V = 151936 in the scratch's 11520 rows: 8192 rows are 256 large logit
    tiles, one for every CU."""
    assert _step()(2048, 4096, 151936, 11520, True, True) == 8192
