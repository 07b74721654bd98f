"""Rules of csrc/lp_kernels.h that say which layers a kernel takes, compiled for the host: what a kernel holds in LDS is enough for every layer
that its rule accepts."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2112_05387_amd", "csrc")

PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <random>
#include "lp_kernels.h"
#define CHECK(c) do { if (!(c)) { std::printf("failed: %s\n", #c); return 1; } } while (0)
using namespace lp;
// the head with the loss: features, means and logits of a sample in the 64 KB that a launch has without asking
static int heads() {
    auto takes = [](int HW, int C, int classes, int esz) { HeadProb p; std::memset(&p, 0, sizeof(p)); p.HW = HW; p.C = C; p.classes = classes; return head_with_loss(p, esz); };
    CHECK(takes(64, 64, 256, 4) && !takes(64, 64, 257, 4) && takes(128, 64, 10, 4) && !takes(129, 64, 10, 4));
    for (int esz : {2, 4})
        for (int C = 16 / esz; C <= 2048; C += 16 / esz)
            for (int HW : {1, 2, 3, 4, 8, 16, 49, 64, 256, 1024})
                for (long classes : {1l, 2l, 10l, 16384l / C, 16384l / C + 1, 65536l, 1l << 20, 1l << 21, (1l << 31) / C, (1l << 32) / C, (1l << 31) - 1}) {
                    if (classes < 1 || classes >= 1l << 31) continue;
                    if (takes(HW, C, (int)classes, esz)) CHECK((long)HW * C * esz + (C + classes) * 4 + 1024 <= 65536);
                }
    return 0;
}
// image-facing layers: the rows that a tile of BM pixels copies fit the window, and every tap that lies in the image is among them
static int windows() {
    std::mt19937 g(1);
    auto pick = [&](std::initializer_list<int> v) { return v.begin()[g() % v.size()]; };
    auto in = [&](int lo, int hi) { return lo + (int)(g() % (unsigned)(hi - lo + 1)); };
    int taken = 0;
    for (int it = 0; it < 40000; ++it) {
        const int R = pick({1, 3, 3, 3, 5}), pad = pick({0, R / 2, R / 2}), st = pick({1, 2, 3, 4}), C = pick({1, 2, 3, 3}), esz = pick({2, 4}), BM = pick({64, 256});
        const int H = in(std::max(1, R - 2 * pad), 40), W = in(std::max(1, R - 2 * pad), 40), N = in(1, 6);
        ConvProb p; std::memset(&p, 0, sizeof(p));
        p.OA = p.OH = (H + 2 * pad - R) / st + 1; p.OB = p.OW = (W + 2 * pad - R) / st + 1;
        p.M = N * p.OA * p.OB; p.Ncol = 16; p.Cin = C; p.IH = H; p.IW = W; p.ntr = p.nts = R; p.Kg = p.ldw = R * R * C;
        p.imul = st; p.omul = 1; p.dhs = p.dws = p.rs = p.ss = 1; p.dh0 = p.dw0 = -pad; p.S = R;
        const int lds = iconv_window(p, BM, esz);
        if (R * R * C > 32 || (long)N * H * W * C * esz % 4) CHECK(lds == 0);
        if (!lds) continue;
        ++taken;
        CHECK(lds <= 24 * 1024 + 16);
        const int per = p.OA * p.OB;
        const long total = (long)N * H * W * C * esz;
        for (int m0 = 0; m0 < p.M; m0 += BM) {
            const int ml = std::min(m0 + BM, p.M) - 1, n0 = m0 / per, a0 = m0 % per / p.OB, n1 = ml / per, a1 = ml % per / p.OB;
            const int lo = std::min(std::max(a0 * st - pad, 0), H - 1), hi = std::min(std::max(a1 * st - pad + R - 1, 0), H - 1);
            const long b0 = (long)(n0 * H + lo) * W * C * esz & ~15l, b1 = std::min(((long)(n1 * H + hi + 1) * W * C * esz + 3) & ~3l, total);
            CHECK(b1 > b0 && (b1 - b0 + 1023) / 1024 * 1024 + 16 <= lds);      // whole wave-loads behind a vector of zeros
            for (int m = m0; m <= ml; m += std::max(1, (ml - m0) / 7)) {
                const int n = m / per, a = m % per / p.OB, b = m % per % p.OB;
                for (int r = 0; r < R; ++r)
                    for (int s = 0; s < R; ++s) {
                        const int ih = a * st - pad + r, iw = b * st - pad + s;
                        if (ih < 0 || ih >= H || iw < 0 || iw >= W) continue;
                        const long o = (long)((n * H + ih) * W + iw) * C * esz;
                        CHECK(b0 <= o && o + C * esz <= b1);
                    }
            }
        }
    }
    CHECK(taken > 10000);
    return 0;
}
int main() { return heads() || windows(); }
"""


def test_lds_of_accepted_layers(tmp_path):
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-w", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
