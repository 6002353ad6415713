"""The LDS layout of the convolution workgroups (host code, no GPU).

A workgroup of a ragged list computes products of different sizes in turn.
Between the last barrier of one and the first of the next, a slow wave still
reads the one's result carries while a fast wave writes the next one's recode
carries; after that first barrier a wave reads recode carries while others
write digits.  Neither pair of areas may overlap, for any two sizes."""
from __future__ import annotations

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHECK = r"""
#include <cstdio>
#include <initializer_list>
#include "conv_layout.hpp"
using namespace bi::conv;
static bool meet(uint32_t p, uint32_t pn, uint32_t q, uint32_t qn) { return p < q + qn && q < p + pn; }
int main() {
    const uint32_t units = 32, waves = 16;
    long bad = kCarryWords + units > kSumWords || kBoundaryWords + units > kCarryWords ||
               kRecodeB + waves > kBoundaryWords || kRecodeWords + waves > kRecodeB;
    for (uint32_t cap : {64, 96, 128, 160, 192, 256, 384, 512, 1024, 2048})  // chunks of the kernels' largest products
        for (uint32_t n = 1; n <= cap; ++n) {
            const WgLayout x = wg_layout(n, cap);
            // digits of a, of b, the exchanged words: in this order and inside the block
            bad += wg_a_bytes(n) > x.b || x.b + wg_b_bytes(n) > x.sum || x.sum + 4 * kSumWords > x.total ||
                   x.total > wg_layout(cap, cap).total;
            for (uint32_t m = 1; m <= cap; ++m) {
                const WgLayout y = wg_layout(m, cap);
                for (uint32_t at : {kRecodeWords, kRecodeB})
                    if (meet(y.sum + 4 * at, 4 * waves, x.sum + 4 * kCarryWords, 4 * units) && bad++ == 0)
                        std::printf("first: %u chunks after %u\n", m, n);
            }
        }
    std::printf("%ld overlaps\n", bad);
    return bad != 0;
}
"""


def test_carry_words_of_successive_products(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "layout.cpp", tmp_path / "layout"
    src.write_text(CHECK)
    subprocess.run([cxx, "-std=c++17", "-O2", "-I", os.path.join(ROOT, "paper_2405_14642_amd", "csrc"), str(src), "-o",
                    str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
