"""The radix sort's workspace, asked of the library on the host: a context that
reserved room for n particles sorts any smaller set without allocating."""
import ctypes as C
import os

import pytest


@pytest.fixture(scope="module")
def words():
    from paper_2511_21921_amd import crk
    if not os.path.exists(crk.LIB_PATH):
        from paper_2511_21921_amd import build
        build.build()
    f = crk.lib()._ZN3crk15radix_tmp_wordsEl  # crk::radix_tmp_words(int64_t)
    f.argtypes, f.restype = [C.c_int64], C.c_int64
    return f


def test_workspace_never_falls_as_the_set_grows(words):
    sizes = sorted({n + d for n in [2048 * k for k in range(1, 4096, 7)] +
                    [1 << b for b in range(0, 26)] for d in (-1, 0, 1)} - {-1, 0})
    got = [words(n) for n in sizes]
    for (n0, a), (n1, b) in zip(zip(sizes, got), zip(sizes[1:], got[1:])):
        assert a <= b, (n0, a, n1, b)


def test_workspace_holds_the_widest_digits(words):
    """A histogram of 2^10 digits per 2048 keys up to 2^20 keys, of 2^8 beyond."""
    for n in (1, 2048, 2049, 1 << 20, (1 << 20) + 1, 2000000, 1 << 24):
        assert words(n) >= (-(-n // 2048)) << (10 if n <= 1 << 20 else 8), n
