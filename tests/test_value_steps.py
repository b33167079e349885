"""The equal steps of the selections' histograms, on the host: a small C++ program includes their header and is stopped by a
conversion to int out of its range."""
from __future__ import annotations

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cmath>
#include <cstdio>
#include <initializer_list>
#include "value_steps.hpp"

// values of [lo, hi] in ascending order: steps ascend and stay in [0, n), the ends in the first and the last one
static int walk(float lo, float hi, int n)
{
    float per_unit;
    if (!sf::cut_range(lo, hi, n, per_unit)) return 0;
    int last = 0;
    for (int i = 0; i <= 5000; ++i) {
        const float v = i == 5000 ? hi : std::fmin(hi, std::fmax(lo, (float)(lo + ((double)hi - lo) * i / 5000)));
        const int s = sf::step_of(v, lo, per_unit, n);
        if (s < last || s >= n || (i == 0 && s) || (i == 5000 && s != n - 1)) return std::printf("%g..%g: step %d of %g after %d\n", lo, hi, s, v, last), -1;
        last = s;
    }
    return 1;
}

int main()
{
    for (int n : {512, 1024}) {
        int cut = 0;
        for (float lo : {0.f, 1.f, -1.f, 1e-38f, -1e-40f, -1e30f, 3e37f})
            for (int e = -149; e < 128; ++e) {
                const int r = walk(lo, lo + std::ldexp(1.f, e), n);
                if (r < 0) return 1;
                cut += r;
            }
        if (cut < 500) return std::printf("only %d ranges\n", cut), 1;
        if (walk(0.f, INFINITY, n) || walk(-INFINITY, 0.f, n) || walk(0.f, NAN, n) || walk(NAN, 1.f, n) || walk(-3e38f, 3e38f, n) || walk(2.f, 2.f, n))
            return std::printf("no range\n"), 1;
        if (walk(0.f, 1e-6f, n) != 1 || walk(-1.f, 1.f, n) != 1) return std::printf("a range\n"), 1;
    }
    return 0;
}
"""


def test_steps_of_every_range(tmp_path):
    src, exe = tmp_path / "steps.cpp", tmp_path / "steps"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-fsanitize=float-cast-overflow", "-fno-sanitize-recover=all",
                    "-I", os.path.join(ROOT, "paper_2604_08971_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
