"""The strip planner (csrc/plan.cpp) on the CPU: every plan covers its matrix
exactly once, stays inside LDS, the ring and the workspace bound, and is
refused where a PCF does not fit."""
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

static void check(const Plan &p, const std::vector<int64_t> &o, int rb, int64_t r0, int64_t r1,
                  int64_t c0, int64_t c1, bool mirrored)
{
    const int64_t lds = kStripSharedBytes +
                        (int64_t)p.strip_waves * strip_wave_bytes(p.strip_pairs, p.strip_cols) +
                        (int64_t)(p.strip_row_recs + p.strip_ring_recs) * rb;
    CHECK(lds <= kStripLdsBytes);
    CHECK(p.strip_pairs <= kStripMaxPairs && p.strip_cols <= kStripMaxCols);
    CHECK(p.strip_waves >= 4 && p.strip_waves <= kStripMaxWaves);
    CHECK(p.sblocks.size() + 1 == p.blocks.size());
    for (size_t b = 0; b + 1 < p.blocks.size(); ++b) {
        const int64_t a = p.blocks[b], e = p.blocks[b + 1];
        CHECK(e > a && e - a <= kStripMaxRows && (e - a) * p.strip_cols <= p.strip_pairs);
        CHECK(o[e] - o[a] + (e - a) * kPad <= p.strip_row_recs);
        CHECK(p.sblocks[b].lo == a && p.sblocks[b].rows == e - a);
        CHECK(p.sblocks[b].rec0 == o[a] + a * kPad &&
              p.sblocks[b].recs == o[e] - o[a] + (e - a) * kPad);
    }
    for (size_t g = 0; g + 1 < p.groups.size(); ++g) {
        const StripGroup a = p.groups[g], b = p.groups[g + 1];
        const int64_t m = b.start - a.start, len = o[b.start] - o[a.start] + m * kPad;
        CHECK(m >= 1 && m <= p.strip_cols && len <= p.strip_ring_recs);
        CHECK((a.size & ((1 << kStripColShift) - 1)) == len && (a.size >> kStripColShift) == m);
        CHECK(a.rec0 == o[a.start] + a.start * kPad);
        CHECK(a.virt % (uint32_t)p.strip_ring_recs + (uint32_t)len <= (uint32_t)p.strip_ring_recs);
        CHECK(b.virt - a.virt >= (uint32_t)len);
    }
    CHECK(p.runs.size() == (size_t)p.ntiles + 1 && p.runs.front() == 0);
    CHECK(p.runs.back() == (int)p.jobs.size());
    for (size_t i = 0; i + 1 < p.runs.size(); ++i)
        CHECK(p.runs[i] < p.runs[i + 1]);
    const int64_t nr = r1 - r0, nc = c1 - c0;
    std::vector<int> seen((size_t)(nr * nc), 0);
    for (const StripJob &j : p.jobs) {
        const Segment &s = p.segs[(size_t)j.seg];
        CHECK(j.g0 < j.g1 && (size_t)j.g1 < p.groups.size());
        CHECK(p.groups[j.g1].virt - p.groups[j.g0].virt < (1u << 29));
        for (int64_t c = p.groups[j.g0].start; c < p.groups[j.g1].start; ++c)
            for (int64_t i = p.blocks[j.block]; i < p.blocks[j.block + 1]; ++i) {
                if (s.type == kSegTriangle && i > c)
                    continue;
                const int64_t ii = s.swap ? c : i, jj = s.swap ? i : c;
                CHECK(ii >= r0 && ii < r1 && jj >= c0 && jj < c1);
                ++seen[(size_t)((ii - r0) * nc + jj - c0)];
                if (s.mirror && ii != jj)
                    ++seen[(size_t)((jj - r0) * nc + ii - c0)];
            }
    }
    if (mirrored)
        for (int x : seen)
            CHECK(x == 1);
}

int main()
{
    std::mt19937 g(1);
    auto U = [&](int64_t a, int64_t b) { return a + (int64_t)(g() % (uint64_t)(b - a + 1)); };
    int strips = 0, tiles = 0;
    for (int it = 0; it < 400; ++it) {
        // a few CUs, so that small matrices are long launches
        const int cus = it % 3 == 0 ? 4 : 1, rb = it & 1 ? 16 : 8;
        const int64_t n = U(1, 700), lo = U(1, it % 5 == 0 ? 1500 : 60);
        const int64_t hi = lo + U(0, it % 4 == 0 ? 900 : 60);
        std::vector<int64_t> o((size_t)n + 1, 0);
        for (int64_t i = 0; i < n; ++i)
            o[i + 1] = o[i] + (U(0, 60) == 0 ? U(1, it % 11 == 0 ? 12000 : 300) : U(lo, hi));
        TileShape sh;
        if (it % 7 == 3) {
            sh.max_block = (int32_t)U(1, 32);
            sh.budget_div = (int32_t)U(2, 8);
        }
        int64_t r0 = 0, r1 = n, c0 = 0, c1 = n;
        const bool win = it % 2 == 1, upper = it % 13 == 0;
        if (win) {
            r0 = U(0, n); r1 = U(r0, n); c0 = U(0, n); c1 = U(c0, n);
        }
        if (r0 == r1 || c0 == c1)
            continue;
        Plan p, q;
        std::string e;
        CHECK(plan_matrix(n, o.data(), rb, false, win, r0, r1, c0, c1, upper, n, sh, p, e, cus));
        CHECK(plan_matrix(n, o.data(), rb, false, win, r0, r1, c0, c1, upper, n, TileShape(), q, e));
        CHECK(!q.strips);
        CHECK(plan_workspace_bytes(p, rb) <= plan_workspace_bound(q, rb));
        (p.strips ? strips : tiles) += 1;
        if (p.strips)
            check(p, o, rb, r0, r1, c0, c1, !upper);
    }
    CHECK(strips > 60 && tiles > 20);
    // a batch: each problem's matrix once, nothing between problems
    std::vector<int64_t> o(1, 0), so = {0, 0, 1, 3, 260, 320, 700}, oo(6, 0);
    for (int i = 0; i < 700; ++i)
        o.push_back(o.back() + U(1, 40));
    for (int b = 0; b + 1 < 6; ++b)
        oo[(size_t)b + 1] = oo[(size_t)b] + (so[b + 1] - so[b]) * (so[b + 1] - so[b]);
    Plan p;
    std::string e;
    CHECK(plan_batched(6, so.data(), oo.data(), o.data(), 700, 16, false, TileShape(), p, e, 1));
    CHECK(p.strips);
    check(p, o, 16, 0, 700, 0, 700, false);
    std::vector<int> seen((size_t)(oo[5] + 380 * 380), 0);
    for (const StripJob &j : p.jobs) {
        const Segment &s = p.segs[(size_t)j.seg];
        for (int64_t c = p.groups[j.g0].start; c < p.groups[j.g1].start; ++c)
            for (int64_t i = p.blocks[j.block]; i < p.blocks[j.block + 1]; ++i)
                if (i <= c) {
                    ++seen[(size_t)(s.obase + (i - s.row0) * s.ldo + c - s.col0)];
                    if (i != c)
                        ++seen[(size_t)(s.obase + (c - s.row0) * s.ldo + i - s.col0)];
                }
    }
    for (int x : seen)
        CHECK(x == 1);
    // small tile plans: smaller blocks on a device of 256 CUs, none where a
    // shape is asked for or the plan is an adjoint's
    for (int64_t n : {2, 31, 33, 200, 450, 3000}) {
        std::vector<int64_t> of(1, 0);
        for (int64_t i = 0; i < n; ++i)
            of.push_back(of.back() + U(10, 100));
        Plan big, cap, shaped, adj0, adj;
        TileShape sh;
        sh.preset = false;
        CHECK(plan_matrix(n, of.data(), 16, false, false, 0, 0, 0, 0, false, n, TileShape(), big, e));
        CHECK(plan_matrix(n, of.data(), 16, false, false, 0, 0, 0, 0, false, n, TileShape(), cap, e, 256));
        CHECK(plan_matrix(n, of.data(), 16, false, false, 0, 0, 0, 0, false, n, sh, shaped, e, 256));
        CHECK(plan_matrix(n, of.data(), 16, true, false, 0, 0, 0, 0, false, n, TileShape(), adj0, e));
        CHECK(plan_matrix(n, of.data(), 16, true, false, 0, 0, 0, 0, false, n, TileShape(), adj, e, 256));
        CHECK(adj.blocks == adj0.blocks && (shaped.strips || shaped.blocks == big.blocks));
        if (cap.strips)
            continue;
        const int64_t nb = (int64_t)cap.blocks.size() - 1;
        CHECK(cap.ntiles == nb * (nb + 1) / 2 && cap.blocks.front() == 0 && cap.blocks.back() == n);
        CHECK(cap.blocks == big.blocks || cap.ntiles <= 169);
        CHECK(n != 200 || cap.blocks.size() > big.blocks.size());
    }
    std::printf("ok %d strip plans, %d tile plans\n", strips, tiles);
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_strip_plans(tmp_path):
    src, exe = tmp_path / "plan_check.cpp", tmp_path / "plan_check"
    src.write_text(HARNESS)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I", CSRC, "-o", str(exe), str(src),
                           os.path.join(CSRC, "plan.cpp")])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
