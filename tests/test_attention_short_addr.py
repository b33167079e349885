"""The reads of the one-launch attention, walked on the host: a small C++ program includes the kernel's own address header."""
from __future__ import annotations

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _run(tmp_path, program):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(program)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2604_08971_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


# every lane, half and tile of every length: 16 bytes inside the lane's own row, and the tile's own chunk where the row has it
V_READS = r"""
#include <cstdio>
#include <initializer_list>
#include "attention_short_addr.hpp"

int main()
{
    for (int L = 2; L <= 2048; L += L < 200 ? 1 : 61) {
        const int Lp = (L + 7) / 8 * 8;
        for (int pad : {0, 8, 64})
            for (int t = 0; t < (L + 31) / 32; ++t)
                for (int p = 0; p < 2; ++p)
                    for (int lane = 0; lane < 64; ++lane) {
                        const int l32 = lane & 31, lhi = lane >> 5, own = t * 64 + p * 32 + lhi * 16;
                        const uint32_t row = (uint32_t)l32 * (Lp + pad) * 2u, off = sf::short_v_off(t, p, l32, lhi, Lp + pad, Lp);
                        if (off < row || off + 16 > row + Lp * 2u || off % 16 || (own + 16 <= Lp * 2 && off != row + own))
                            return std::printf("L %d tile %d half %d lane %d: %u in a row at %u\n", L, t, p, lane, off, row), 1;
                    }
    }
    return 0;
}
"""


def test_values_are_read_inside_their_row(tmp_path):
    _run(tmp_path, V_READS)
