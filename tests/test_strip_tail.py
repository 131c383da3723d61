"""The strip planner's bound on a long column's item (csrc/plan.cpp), on the CPU:
in every strip plan of short PCFs with a few long ones among them, no item of a
column takes its wave longer than 0.3 of what the launch gives every wave (a pair
counted with 64 steps more): by smaller row blocks, or by no strip plan."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2404_07183_amd", "csrc")

HARNESS = r"""
#include "plan.hpp"
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>
using namespace pcf;
#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); std::exit(1); } } while (0)

int main()
{
    std::mt19937 g(2);
    auto U = [&](int64_t a, int64_t b) { return a + (int64_t)(g() % (uint64_t)(b - a + 1)); };
    int small = 0, full = 0, tiles = 0;
    for (int it = 0; it < 300; ++it) {
        const int cus = 16, rb = it & 1 ? 16 : 8;
        const int64_t n = U(500, 1500), rows = U(10, 60), every = U(20, 600);
        const int64_t many = U(100, it % 3 == 0 ? 3000 : 800);
        std::vector<int64_t> o((size_t)n + 1, 0);
        for (int64_t i = 0; i < n; ++i)
            o[i + 1] = o[i] + (U(0, every) == 0 ? many : U(1, rows));
        const bool win = it % 4 == 1;
        const int64_t r1 = win ? n / 3 : n, c0 = win ? n / 3 : 0;
        Plan p;
        std::string e;
        CHECK(plan_matrix(n, o.data(), rb, false, win, 0, r1, c0, n, false, n, TileShape(), p, e,
                          cus));
        if (!p.strips) {
            ++tiles;
            continue;
        }
        const double mean = (double)o[n] / n;
        const double pairs = win ? (double)r1 * (n - c0) : 0.5 * n * (n + 1);
        const double given = pairs / (64.0 * cus * 16) * (2.0 * mean + 64.0);
        int most = 0;
        for (const StripJob &j : p.jobs) {
            const int64_t R = p.sblocks[j.block].rows;
            most = std::max(most, (int)R);
            const bool tri = p.segs[(size_t)j.seg].type == kSegTriangle;
            for (int k = j.g0; k < j.g1; ++k) {
                const int64_t c = p.groups[k].start, d = p.groups[k + 1].start;
                if (tri && c < 64)
                    continue;
                for (int64_t i = c; i < d; ++i)
                    if (mean < 100.0)
                        CHECK((double)(R * (o[i + 1] - o[i])) / 64.0 <= 0.3 * given * 1.001);
            }
        }
        (most < 64 ? small : full) += 1;
    }
    CHECK(small > 20 && full > 20 && tiles > 20);
    std::printf("ok %d small, %d full, %d tiles\n", small, full, tiles);
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_long_columns(tmp_path):
    src, exe = tmp_path / "tail_check.cpp", tmp_path / "tail_check"
    src.write_text(HARNESS)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I", CSRC, "-o", str(exe), str(src),
                           os.path.join(CSRC, "plan.cpp")])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
