"""The operand loads of the tiled GEMM kernels, walked on the host: a small C++ program includes the kernels' own address
header and visits every 16-byte request of every tile."""
from __future__ import annotations

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "gemm_tile_addr.hpp"

// rows of A, K, row stride, tile rows; mapped: rows are read through a map that reverses them
static int walk(int64_t rows, int K, int64_t ld, int bm, bool mapped)
{
    const int64_t end = ((rows - 1) * ld + K) * 2;                     // bytes of the operand from row 0
    std::vector<int32_t> map;
    for (int64_t i = 0; i < rows; ++i) map.push_back((int32_t)(rows - 1 - i));
    int cut = 0;
    for (int64_t m0 = 0; m0 < rows; m0 += bm) {
        const int64_t base = mapped ? 0 : m0 * ld * 2;
        const uint32_t n = sf::records(mapped ? rows : rows - m0, ld, K);
        if (base + (int64_t)n != end) return std::printf("records end at %lld, operand at %lld\n", (long long)(base + n), (long long)end), 1;
        const int tile_rows = (int)(rows - m0 < bm ? rows - m0 : bm);
        for (int sr4 = 0; sr4 < bm / 8; ++sr4)
            for (int lane = 0; lane < 64; ++lane) {
                const uint32_t off = sf::lane_off(sr4, lane, tile_rows, ld, mapped ? map.data() + m0 : nullptr);
                const int chunk = (int)(off / 2 % ld % 64 / 8);
                for (int kt = 0; kt * 64 < K; ++kt) {
                    const int64_t at = (int64_t)off + kt * 128;
                    if (at + 16 <= (int64_t)n) continue;
                    ++cut;                                              // must lie behind the operand as a whole, and in the K tail
                    if (at < (int64_t)n || kt * 64 + chunk * 8 < K)
                        return std::printf("rows %lld K %d: request at %lld of %u is needed\n", (long long)rows, K, (long long)at, n), 1;
                }
            }
    }
    if (K % 64 && ld == K && cut == 0) return std::printf("rows %lld K %d: no request of the tail was cut\n", (long long)rows, K), 1;
    return 0;
}

int main()
{
    for (int64_t rows : {1, 31, 32, 33, 127, 128, 129, 300})
        for (int K : {64, 96, 128, 160, 352})
            for (int pad : {0, 64})
                for (int bm : {32, 64, 128})
                    for (bool mapped : {false, true})
                        if (walk(rows, K, K + pad, bm, mapped)) return 1;
    return 0;
}
"""


def test_no_request_behind_the_operand(tmp_path):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2604_08971_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
