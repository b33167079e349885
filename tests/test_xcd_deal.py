"""How masked attention problems are dealt to the XCDs, on the host."""
from __future__ import annotations

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# every problem once; and with every second sample costly (or every fourth, with eights enough) half (a quarter) of an XCD's problems are
PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include <vector>
#include "xcd_deal.hpp"

int main()
{
    for (int nG : {1, 2, 3, 4, 8, 12})
        for (int B : {8, 16, 24, 32, 64, 128}) {
            const int n = B * nG, per = n / 8;
            std::vector<int> seen(n, 0);
            for (int x = 0; x < 8; ++x) {
                int second = 0, fourth = 0;
                for (int j = 0; j < per; ++j) {
                    const int p = sf::deal(x, j);
                    if (p < 0 || p >= n) return std::printf("%d of %d\n", p, n), 1;
                    ++seen[p];
                    second += p / nG % 2 == 0;
                    fourth += p / nG % 4 == 0;
                }
                const bool whole = 8 % nG == 0;                           // the groups of a sample within one eight
                if (whole && (2 * second > per + 1 || 2 * second < per - 1))
                    return std::printf("B %d nG %d XCD %d: %d of %d\n", B, nG, x, second, per), 1;
                if (whole && per % 8 == 0 && 4 * fourth != per) return std::printf("B %d nG %d XCD %d: %d of %d\n", B, nG, x, fourth, per), 1;
            }
            for (int p = 0; p < n; ++p)
                if (seen[p] != 1) return std::printf("problem %d of %d: %d times\n", p, n, seen[p]), 1;
        }
    return 0;
}
"""


def test_costly_samples_are_spread(tmp_path):
    src, exe = tmp_path / "deal.cpp", tmp_path / "deal"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2604_08971_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
