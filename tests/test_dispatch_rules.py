"""Which products a single call runs (the library's own rules, which need no GPU): the
shapes whose results the GPU tests compare between kernels do take the kernel they are
named for, and the rules turn where they say."""
import ctypes

import pytest

import paper_2512_08321_amd as ozc
from test_gpu_64_tiles import test_equal_to_128_tiles as tiles_test
from test_gpu_k_split import test_parts_equal_whole as parts_test
from test_gpu_random_calls import NEARLY_FULL

CUS = 256


@pytest.fixture(scope="module")
def rules():
    L = ctypes.CDLL(ozc.library_path)
    # ozc::choose_64_tiles(int, int, long, long, long, int), ozc::choose_k_split(int x 3, long x 3, int)
    t64 = L._ZN3ozc15choose_64_tilesEiillli
    t64.restype, t64.argtypes = ctypes.c_bool, [ctypes.c_int] * 2 + [ctypes.c_int64] * 3 + [ctypes.c_int]
    split = L._ZN3ozc14choose_k_splitEiiillli
    split.restype, split.argtypes = ctypes.c_uint64, [ctypes.c_int] * 3 + [ctypes.c_int64] * 3 + [ctypes.c_int]

    def choose(t, m, n, k, N, algo):
        tile = 256 if m >= 1024 and n >= 1024 else 128
        up = lambda x, a: (x + a - 1) // a * a
        form = 2 if t in "ds" else int(algo == "4m")
        r = split(tile, form, N, up(m, tile), up(n, tile), up(k, 64), CUS)
        parts, first = r >> 32, r & 0xffffffff
        cut = parts > 1 and first < N
        return "parts" if cut else ("64" if t64(tile, N, m, n, up(k, 64), CUS) else "whole")

    return choose


def _cases(test):
    return [mark.args[1] for mark in test.pytestmark if mark.name == "parametrize"][0]


def test_shapes_of_the_kernel_comparisons(rules):
    for t, m, n, k, N, algo in _cases(tiles_test) + [NEARLY_FULL]:
        # one of the list is cut along k; NEARLY_FULL is its neighbour that is not
        want = "parts" if (m, k, algo) == (256, 512, "4m") else "64"
        assert rules(t, m, n, k, N, algo) == want, (t, m, n, k, N)
    for t, m, n, k, N, _, algo in _cases(parts_test):
        assert rules(t, m, n, k, N, algo) == "parts", (t, m, n, k, N)


def test_where_64_tiles_end(rules):
    # 640 blocks of 64 x 64 (2.5 a CU) up to k = 1024, 256 beyond
    assert rules("z", 640, 512, 1024, 8, "karatsuba") == "64"
    assert rules("z", 641, 512, 1024, 8, "karatsuba") == "whole"
    assert rules("z", 640, 512, 1025, 8, "karatsuba") == "whole"
    assert rules("d", 256, 512, 1025, 8, "karatsuba") == "64"
    assert rules("d", 257, 512, 1025, 8, "karatsuba") != "64"
    assert rules("z", 2048, 2048, 64, 2, "karatsuba") != "64"
