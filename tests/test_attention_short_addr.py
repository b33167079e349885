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


# partial results, keys and the context vector are read and written 16 bytes at a time; the pieces do not overlap
LAYOUT = r"""
#include <cstdio>
#include "attention_short_addr.hpp"

template <int DH, int NW> int check()
{
    for (int L = 2; L <= 2048; ++L)
        for (int U = 1; U < L && U < NW * 32; U += U < 40 ? 1 : 37) {
            const sf::ShortLds<DH, NW> a(L, U);
            const size_t nt = (L + 31) / 32, at[] = {a.keys_at, a.ml, a.sel_keys, a.qmax, a.words, a.rows, a.red, a.kbar, a.ctx, a.bytes},
                         need[] = {nt * 32 * DH * 2, NW * 32 * 4, (size_t)L * 4, (size_t)L * 4, nt * 4, (size_t)(U > 64 ? U : 64) * 4,
                                   NW * (DH > 32 ? DH : 32) * 4, DH * 4, DH * 2};
            for (int i = 0; i < 9; ++i)
                if (at[i] + need[i] > at[i + 1]) return std::printf("dh %d waves %d L %d U %d: piece %d\n", DH, NW, L, U, i), 1;
            if (a.ml < (size_t)NW * 32 * DH * 4 || a.keys_at % 16 || a.ctx % 16) return std::printf("dh %d waves %d L %d U %d: %zu\n", DH, NW, L, U, a.ctx), 1;
        }
    return 0;
}

int main() { return check<32, 4>() || check<32, 8>() || check<32, 16>() || check<64, 4>() || check<64, 8>() || check<64, 16>(); }
"""


def test_layout_is_aligned(tmp_path):
    _run(tmp_path, LAYOUT)
