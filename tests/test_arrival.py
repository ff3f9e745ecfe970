"""The counters by which the last work-group of a launch tells the host that everything is there (csrc/arrival.h), on the CPU: the last one
alone is told, and the counters are zero by then without a store that could still be on its way, for whoever hears of it may hand them
to another launch."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "arrival.h"
#include <algorithm>
#include <cstdio>
#include <random>
#include <vector>
using namespace fscnn;
static int counters[kCounterInts];
struct Mem {
    int count(int *p, int most) const { const int was = *p; *p = was >= most ? 0 : was + 1; return was; }
};
int main()
{
    std::mt19937 rng(1);
    for (int groups = 1; groups <= 70; ++groups)
        for (int round = 0; round < 20; ++round) {
            std::vector<int> order(groups);
            for (int i = 0; i < groups; ++i) order[i] = i;
            std::shuffle(order.begin(), order.end(), rng);
            int told = 0;
            for (int i = 0; i < groups; ++i)
                if (arrive(Mem(), counters, groups, order[i])) {
                    ++told;
                    if (i != groups - 1) { std::printf("%d groups: told after %d\n", groups, i + 1); return 1; }
                }
            if (told != 1) { std::printf("%d groups: told %d times\n", groups, told); return 1; }
            for (int c : counters)
                if (c) { std::printf("%d groups: a counter is handed on at %d\n", groups, c); return 1; }
        }
    return 0;
}
"""


def test_counters_are_zero_when_the_last_one_is_told(tmp_path):
    src, exe = tmp_path / "arrival.cpp", tmp_path / "arrival"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_2212_08815_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
