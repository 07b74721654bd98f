"""Which form of the narrow filter-gradient kernel takes a layer (csrc/lp_fwform.h), compiled for the host: the columns that the
form writes are the layer's own, at every width and filter size that the kernel takes."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2112_05387_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "lp_fwform.h"
#define CHECK(c) do { if (!(c)) { std::printf("failed: %s (%d -> %d channels, %d x %d)\n", #c, cin, cout, R, R); bad = 1; } } while (0)
template <int ESZ> static int forms() {
    int bad = 0;
    for (int cin : {1, 2, 3, 16, 32, 64})
        for (int cout : {16, 32, 64})
            for (int R : {1, 3}) {
                if (cin < 16 && R != 3) continue;
                int calls = 0, taps = 0;
                bool stem = false, sixteen = false;
                lp::fwgrad_form<ESZ>(cin, cout, R, [&](auto n, auto s, auto w) { ++calls; taps = decltype(n)::value; stem = decltype(s)::value; sixteen = decltype(w)::value; });
                CHECK(calls == 1);
                CHECK(stem == (cin < 16));
                if (stem) CHECK(taps * 16 >= R * R * cin);      // groups of 16 of the R * R * cin columns
                else CHECK(taps == R * R);                      // a tap a group: no column that the filter does not have
                CHECK(sixteen == (ESZ == 4 && cin == 16 && cout == 16 && R == 3));
            }
    return bad;
}
int main() { return forms<2>() | forms<4>(); }
"""


def test_every_layer_has_its_own_columns(tmp_path):
    src, exe = tmp_path / "form.cpp", tmp_path / "form"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
