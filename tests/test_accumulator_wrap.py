"""Sums and differences of INT32 accumulators (csrc/acc_math.h) at the ends of their range:
defined modulo 2^32.  Evaluated by the compiler as constants, where signed overflow is an
error, and at run time under the undefined-behaviour sanitizer."""
import os
import subprocess

HARNESS = r"""
#include <climits>
#include <cstdio>
#include "acc_math.h"
using namespace ozc;
static_assert(acc_sub(INT_MIN, 1) == 0x7fffffffu, "");
static_assert(acc_sub(127, INT_MIN) == 0x8000007fu, "");
static_assert(acc_add(INT_MAX, 127) == 0x8000007eu, "");
static_assert(acc_add(INT_MIN, INT_MIN) == 0u, "");
static_assert(acc_sub(acc_sub(INT_MAX, INT_MIN), INT_MIN) == INT_MAX, "");
static_assert(acc_flip(INT_MIN) == 0u && acc_flip(-1) == 0x7fffffffu, "");
static_assert(acc_refill(0, true) == 0x7fffff80 && acc_refill(0, false) == -128, "");
static_assert(acc_refill(255, true) == kAccBias + 127, "");
int main() {
    const int v[] = {INT_MIN, INT_MIN + 1, -16129, -1, 0, 1, 127, 16129, INT_MAX - 127, INT_MAX};
    for (int volatile a : v)
        for (int volatile b : v) {
            const long long s = (long long)a + b, d = (long long)a - b;
            if (acc_add(a, b) != (uint32_t)s || acc_sub(a, b) != (uint32_t)d) return 1;
            if (acc_flip(a) != (uint32_t)((long long)a + (1ll << 31))) return 2;
        }
    for (uint32_t u = 0; u < 256; ++u)
        if ((uint32_t)acc_refill(u, true) != u - 128 + (1u << 31) || acc_refill(u, false) != (int)u - 128) return 3;
    puts("ok");
}
"""


def test_wrap(tmp_path):
    csrc = os.path.join(os.path.dirname(__file__), "..", "paper_2512_08321_amd", "csrc")
    (tmp_path / "h.cpp").write_text(HARNESS)
    exe = str(tmp_path / "h")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-O1", "-fsanitize=undefined",
                    "-fno-sanitize-recover=all", "-I" + csrc, str(tmp_path / "h.cpp"), "-o", exe], check=True)
    assert subprocess.run([exe], capture_output=True, text=True, check=False).stdout == "ok\n"
