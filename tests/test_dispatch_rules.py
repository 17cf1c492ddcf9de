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
        form = 2 if t in "ds" else int(algo == "4m")
        k_pad = (k + 63) // 64 * 64
        r = split(tile, form, N, m, n, k_pad, CUS)
        parts, first = r >> 32, r & 0xffffffff
        small = t64(tile, N, m, n, k_pad, CUS)
        return "parts" if parts > 1 and first < N else ("64" if small else "whole"), small

    return choose


def _cases(test):
    return [mark.args[1] for mark in test.pytestmark if mark.name == "parametrize"][0]


def test_shapes_of_the_kernel_comparisons(rules):
    for t, m, n, k, N, algo in _cases(tiles_test) + [NEARLY_FULL]:
        assert rules(t, m, n, k, N, algo)[0] == "64", (t, m, n, k, N)
    for t, m, n, k, N, _, algo in _cases(parts_test):
        assert rules(t, m, n, k, N, algo)[0] == "parts", (t, m, n, k, N)


def test_where_64_tiles_end(rules):
    # 640 blocks of 64 x 64 (2.5 a CU) up to k = 1024, 256 beyond
    for shape, small in (((640, 512, 1024), True), ((641, 512, 1024), False), ((640, 512, 1025), False),
                         ((256, 512, 1025), True), ((257, 512, 1025), False), ((2048, 2048, 64), False)):
        assert rules("z", *shape, 8, "karatsuba")[1] == small, shape


def test_short_parts_do_not_pay(rules):
    """Calls of a few slabs that ran up to a third longer cut than whole."""
    for case in (("z", 47, 110, 791, 11, "karatsuba"), ("z", 256, 256, 512, 14, "4m"), ("c", 366, 65, 326, 10, "4m"),
                 ("d", 80, 136, 2022, 14, "karatsuba"), ("c", 179, 128, 1146, 16, "karatsuba")):
        assert rules(*case)[0] != "parts", case
    for case in (("z", 384, 320, 40000, 14, "karatsuba"), ("z", 21, 21, 24942, 13, "karatsuba"),
                 ("c", 169, 96, 6215, 6, "4m"), ("z", 2048, 2048, 2048, 13, "karatsuba")):
        assert rules(*case)[0] == "parts", case
