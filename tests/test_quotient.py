"""The division by the sampling temperature (csrc/quotient.hpp), on the host:
the same plain C++ the kernels compile, against the host's own IEEE division."""
from __future__ import annotations

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <random>
#include "quotient.hpp"

static float bits(uint32_t u) { float x; std::memcpy(&x, &u, 4); return x; }

int main()
{
    // divisors: the mantissas next to a power of two and random ones, over the
    // exponents of [kQuotientLo, kQuotientHi], both ends included
    std::mt19937 rng(20);
    const uint32_t edge[] = {0x7FFFFF, 0x7FFFFE, 1, 2, 0x400000, 0x3FFFFF, 0x400001, 0};
    long bad = 0;
    for (int k = 0; k < 24; ++k) {
        const uint32_t m = k < 8 ? edge[k] : rng() & 0x7FFFFF;
        const float b = k == 22 ? roi::kQuotientLo : k == 23 ? roi::kQuotientHi
                        : bits((107 + (k * 7) % 40) << 23 | m);
        const float y = (float)(1.0 / (double)b);
        // every mantissa of the dividend, at exponents from 2^-100 to 2^99
        const uint32_t e = k % 3 == 0 ? 27 : k % 3 == 1 ? 226 : 127;
        for (uint32_t a = 0; a < (1u << 23); ++a) {
            const float x = bits(e << 23 | a);
            bad += roi::quotient(x, b, y) != x / b;
            bad += roi::quotient(-x, b, y) != -x / b;
        }
        bad += roi::quotient(0.0f, b, y) != 0.0f;
        bad += roi::quotient(roi::kQuotientMax, b, y) != roi::kQuotientMax / b;
    }
    std::printf("%ld\n", bad);
    return 0;
}
"""


def test_quotient_is_the_ieee_division(tmp_path):
    src, exe = tmp_path / "q.cpp", tmp_path / "q"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-O2", "-mfma", "-ffp-contract=off", "-std=c++17",
                    "-I" + os.path.join(ROOT, "paper_2608_23048_amd", "csrc"), str(src), "-o",
                    str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=120)
    assert out.stdout.strip() == "0", f"{out.stdout.strip()} quotients differ from the division"
