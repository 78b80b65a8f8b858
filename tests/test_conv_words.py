"""The two forms in which the lowered-convolution kernels find their operand
words -- every word's position divided out, or carried from slab to slab --
compared word for word on the CPU: kernels, strides, paddings and channel
counts (multiples of 4), pieces that start and end anywhere, both operand
orders and both register tiles.  Compiled with bounds checks: neither form may
read outside the input."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1812_08011_amd", "csrc")

PROGRAM = r"""
#define __device__
#define __forceinline__ inline
#include "gemm_conv_words.h"
#include <cstdio>
#include <cstdlib>
#include <vector>
using namespace fp8t;
using namespace fp8t::valu_impl;

template <bool KC, int R, int BK, int NT, int W>
bool same(int it) {
    ConvGeom g{};
    g.C = 4 * (1 + rand() % (it % 3 ? 12 : 40));
    g.H = 1 + rand() % 9; g.W = 1 + rand() % 9;
    const int KH = 1 + rand() % 5;
    g.KW = 1 + rand() % 5; g.pad = rand() % 4; g.stride = 1 + rand() % 3; g.vec = 1;
    if (g.H + 2 * g.pad < KH || g.W + 2 * g.pad < g.KW) return true;
    const int OH = (g.H + 2 * g.pad - KH) / g.stride + 1;
    g.OW = (g.W + 2 * g.pad - g.KW) / g.stride + 1;
    g.OHW = OH * g.OW; g.KWC = g.KW * g.C;
    const int N = 1 + rand() % 6, M = N * g.OHW, K = KH * g.KWC;
    std::vector<uint8_t> X((size_t)N * g.H * g.W * g.C);
    for (auto& x : X) x = (uint8_t)(1 + rand() % 255);
    const int rows = KC ? M : K, len = KC ? K : M;
    const int r0 = rand() % ((rows + R - 1) / R) * R;
    const int kbeg = KC ? rand() % (len / 4) * 4 : rand() % len;
    const int kend = kbeg + 1 + rand() % (len - kbeg);
    for (int t = 0; t < NT; ++t) {
        ConvWalk<KC, R, BK, NT, W> walk;
        walk.start(g, r0, kbeg, t);
        for (int k = kbeg; k < kend; k += BK) {
            uint32_t a[W], b[W];
            walk.load(X.data(), g, r0, rows, k, kend, t, a);
            slab_load_conv<KC, R, BK, NT, W>(X.data(), g, r0, rows, k, kend, t, b);
            for (int w = 0; w < W; ++w)
                if (a[w] != b[w]) {
                    printf("KC %d C %d H %d W %d KW %d pad %d stride %d r0 %d k %d..%d thread %d\n",
                           KC, g.C, g.H, g.W, g.KW, g.pad, g.stride, r0, k, kend, t);
                    return false;
                }
        }
    }
    return true;
}

int main() {
    srand(3);
    for (int it = 0; it < 600; ++it)
        if (!same<true, 64, 32, 256, 2>(it) || !same<false, 64, 32, 256, 2>(it) ||
            !same<true, 128, 32, 512, 2>(it) || !same<false, 128, 32, 512, 2>(it))
            return 1;
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ needed")
def test_carried_positions_give_the_divided_ones(tmp_path):
    src, exe = tmp_path / "words.cpp", tmp_path / "words"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-fsanitize=address,undefined",
                           "-fno-sanitize-recover=all", "-I", CSRC, "-o", str(exe), str(src)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
