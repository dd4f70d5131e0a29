"""Division by a number that the host knows (csrc/divisor.h), compiled for the host: exact over the range that it was asked for."""
import ctypes as C
import os
import random
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_2209_09130_amd", "csrc")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("divisor")
    (d / "d.cpp").write_text('#include "divisor.h"\n'
                             'extern "C" unsigned divisor(unsigned long long n, unsigned d) { return samp::divisor(n, d); }\n'
                             'extern "C" unsigned over(unsigned n, unsigned by, unsigned d) { return samp::over(n, by, d); }\n')
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(d / "d.so"), str(d / "d.cpp")], check=True)
    lib = C.CDLL(str(d / "d.so"))
    lib.divisor.argtypes, lib.divisor.restype = [C.c_ulonglong, C.c_uint], C.c_uint
    lib.over.argtypes, lib.over.restype = [C.c_uint, C.c_uint, C.c_uint], C.c_uint
    return lib


@pytest.mark.parametrize("n", [1, 2, 12, 257, 4096, 65537, 1 << 24, (1 << 25) + 1, (1 << 32) - 1])
def test_quotients_are_exact_below_n(lib, n):
    rnd = random.Random(n)
    for d in [*range(1, 140), 144, 768, 1536, 3072, 4095, 4096, 4097, 65535, 65536, 1 << 20, (1 << 31) - 1]:
        by = lib.divisor(n, d)
        top = n // d
        xs = {0, n - 1, *(v for q in (1, 2, top // 2, top - 1, top) for v in (q * d - 1, q * d)), *(rnd.randrange(n) for _ in range(20))}
        for x in xs:
            if 0 <= x < n:
                assert lib.over(x, by, d) == x // d, (n, d, x)


def test_sizes_of_ordinary_batches_need_no_division(lib):
    """Strips of 32 queries per sequence, heads, and tiles of a GEMM, for 65536 tokens and for the largest batch."""
    for items in (65536 // 32 * 32, (1 << 24) // 32 * 32):
        assert all(lib.divisor(items, d) > 1 for d in [*range(2, 129)])
    assert lib.divisor(1 << 24, 1) == 0 and lib.divisor((1 << 32) - 1, 12) == 1
