"""The launchers' per-device setup (csrc/lp_once.h), compiled for the host: every device gets it, from whichever thread
launches there first, and a failure is not remembered as done."""
import glob
import os
import re
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2112_05387_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <thread>
#include <vector>
#include "lp_once.h"
static thread_local int current = 0;
static std::atomic<int> calls[80];
static std::atomic<int> fail{0};
static int get(int* d) { *d = current; return current == 79 ? 7 : 0; }
static int work() { if (fail.load()) return 3; ++calls[current]; return 0; }
#define CHECK(c) do { if (!(c)) { std::printf("failed: %s\n", #c); return 1; } } while (0)
int main() {
    lp::OncePerDevice once;
    fail = 1; CHECK(once.run(get, work) == 3);
    fail = 0; CHECK(once.run(get, work) == 0 && calls[0] == 1);
    CHECK(once.run(get, work) == 0 && calls[0] == 1);
    for (int d : {1, 63}) { current = d; once.run(get, work); once.run(get, work); CHECK(calls[d] == 1); }
    current = 64; once.run(get, work); once.run(get, work); CHECK(calls[64] == 2);
    current = 79; CHECK(once.run(get, work) == 7 && calls[79] == 0);
    std::vector<std::thread> t;
    for (int i = 0; i < 8; ++i) t.emplace_back([&once, i] { current = 8 + i % 4; for (int k = 0; k < 1000; ++k) once.run(get, work); });
    for (auto& x : t) x.join();
    for (int d = 8; d < 12; ++d) CHECK(calls[d] >= 1 && calls[d] <= 2);
    return 0;
}
"""


def test_once_per_device(tmp_path):
    src, exe = tmp_path / "once.cpp", tmp_path / "once"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=thread", "-pthread", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr


def test_launchers_keep_no_flag_of_their_own():
    for path in glob.glob(os.path.join(CSRC, "*.hip")):
        assert not re.search(r"static bool \w+ = false", open(path).read()), path
