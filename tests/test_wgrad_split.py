"""How a launch of the wide filter-gradient kernel is dealt to the XCDs and cut into pieces (csrc/lp_wgsplit.h), compiled for
the host: every piece goes to exactly one workgroup, no XCD has two more than another, consecutive pieces share an XCD."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2112_05387_amd", "csrc")

PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "lp_wgsplit.h"
#define CHECK(c) do { if (!(c)) { std::printf("failed: %s\n", #c); return 1; } } while (0)
using namespace lp;
static int deal(const std::vector<int>& n) {
    int total = 0;
    for (int v : n) total += v;
    const int grid = xcd_grid(total), np = (int)n.size();
    std::vector<std::vector<int>> at(np);
    for (int i = 0; i < np; ++i) at[i].assign(n[i], -1);
    std::vector<int> per(8, 0);
    for (int b = 0; b < grid; ++b) {
        int prob = -1, local = -1;
        if (!xcd_piece(b, np, [&](int i) { return n[i]; }, prob, local)) continue;
        CHECK(prob >= 0 && prob < np && local >= 0 && local < n[prob] && at[prob][local] < 0);
        at[prob][local] = b & 7;
        ++per[b & 7];
    }
    int lo = 1 << 30, hi = 0;
    for (int v : per) { lo = v < lo ? v : lo; hi = v > hi ? v : hi; }
    CHECK(hi - lo <= 1);
    for (int i = 0; i < np; ++i) {
        int changes = 0;
        for (int j = 0; j < n[i]; ++j) { CHECK(at[i][j] >= 0); changes += j && at[i][j] != at[i][j - 1]; }
        CHECK(changes <= 7);
    }
    return 0;
}
// cost of a plan without a rest, and the lowest of any
static double cost_of(const SplitPart* p, int n, const SplitCost& c, int chunk) {
    long blocks = 0;
    bool whole = true;
    for (int i = 0; i < n; ++i) { const int ks = (p[i].kt + chunk - 1) / chunk; blocks += (long)p[i].tiles * ks; whole = whole && ks == 1; }
    return (double)((blocks + c.slots - 1) / c.slots) * c.round(chunk, whole);
}
static int full_group(int tiles, int kt, const SplitCost& c) {
    SplitPart p[16];
    for (auto& q : p) q = {tiles, kt, 0};
    int s = 0;
    CHECK(plan_wgrad_pieces(p, 16, s, c, 16, false) == 0);
    double best = 1e300;
    for (int chunk = 16; chunk <= kt; ++chunk) best = std::min(best, cost_of(p, 16, c, chunk));
    CHECK(cost_of(p, 16, c, (kt + p[0].ksplit - 1) / p[0].ksplit) <= best);
    return 0;
}
// the same plan as a search through every length
static int every_length(SplitPart* p, int n, const SplitCost& c, int min_chunk, bool may_cut) {
    SplitPart q[16];
    int max_kt = 1, best_chunk = min_chunk, rest = 0, rest_split = 1, s = 0;
    double best = 1e300;
    for (int i = 0; i < n; ++i) { q[i] = p[i]; max_kt = std::max(max_kt, p[i].kt); }
    for (int chunk = min_chunk; chunk <= std::max(max_kt, min_chunk); ++chunk) {
        long blocks = 0;
        bool whole = true;
        for (int i = 0; i < n; ++i) { const int ks = (p[i].kt + chunk - 1) / chunk; blocks += (long)p[i].tiles * ks; whole = whole && ks == 1; }
        const double cost = cost_of(p, n, c, chunk);
        if (cost < best) { best = cost; best_chunk = chunk; rest = 0; rest_split = 1; }
        const int over = (int)(blocks % c.slots), cut = over ? c.slots / over : 1;
        if (!may_cut || !whole || blocks < c.slots || cut < 2 || over >= p[n - 1].tiles || p[n - 1].kt / cut < 8) continue;
        const double two = (double)(blocks / c.slots) * c.round(chunk, true) + c.round((p[n - 1].kt + cut - 1) / cut, false);
        if (two < best) { best = two; best_chunk = chunk; rest = over; rest_split = cut; }
    }
    CHECK(plan_wgrad_pieces(q, n, s, c, min_chunk, may_cut) == rest && (!rest || s == rest_split));
    for (int i = 0; i < n; ++i) CHECK(q[i].ksplit == (p[i].kt + best_chunk - 1) / best_chunk);
    return 0;
}
int main() {
    for (int t = 0; t < 600; ++t) {
        SplitPart p[16];
        const int n = 1 + std::rand() % 16, kt = 1 + std::rand() % 4200;
        for (int i = 0; i < n; ++i) p[i] = {1 + std::rand() % 60, t % 3 == 0 ? kt : 1 + std::rand() % (t % 3 == 1 ? 300 : 4200), 0};
        CHECK(!every_length(p, n, t % 2 ? kFastCost : kTileCost, t % 2 ? 16 : 4, t % 5 != 0));
    }
    // no entry for a rest: the best plan that needs none (with one, 17 tiles of 1024 units are whole, and 16 of the 272 are the rest)
    CHECK(!full_group(17, 1024, kFastCost) && !full_group(17, 512, kFastCost) && !full_group(33, 1024, kFastCost) && !full_group(33, 700, kTileCost));
    std::srand(1);
    CHECK(!deal({51, 51, 51, 51, 51}) && !deal({1}) && !deal({7, 9, 0, 8}) && !deal({255}) && !deal({256, 32}));
    for (int t = 0; t < 300; ++t) {
        std::vector<int> n(1 + std::rand() % 16);
        for (int& v : n) v = std::rand() % 80;
        CHECK(!deal(n));
    }
    for (int t = 0; t < 300; ++t) {                // the plan: pieces that cover every reduction, a rest inside the last problem
        SplitPart p[16];
        const int n = 1 + std::rand() % 16;
        for (int i = 0; i < n; ++i) p[i] = {1 + std::rand() % 60, 1 + std::rand() % (t % 2 ? 4200 : 300), 0};
        int s = 0;
        const int rest = plan_wgrad_pieces(p, n, s);
        for (int i = 0; i < n; ++i) CHECK(p[i].ksplit >= 1 && p[i].ksplit <= p[i].kt);
        CHECK(rest >= 0 && rest < p[n - 1].tiles && (!rest || (s >= 2 && p[n - 1].ksplit == 1 && rest * s <= 256)));
    }
    SplitPart a[6];                                // 288 whole tiles: 256 in one round, the other 32 cut into eight
    for (auto& q : a) q = {48, 256, 0};
    int s = 0;
    CHECK(plan_wgrad_pieces(a, 6, s) == 32 && s == 8 && a[0].ksplit == 1);
    SplitPart b[5];                                // five problems of three long tiles: one round
    for (auto& q : b) q = {3, 4096, 0};
    CHECK(plan_wgrad_pieces(b, 5, s) == 0 && b[0].ksplit == 17);
    return 0;
}
"""


def test_split_and_deal(tmp_path):
    src, exe = tmp_path / "split.cpp", tmp_path / "split"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-fsanitize=undefined,address", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
