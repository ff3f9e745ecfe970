"""The counters by which the last work-group of a launch tells the host that everything is there (csrc/arrival.h), on the CPU with a memory
whose plain stores take effect as late as they may: whoever hears of it may hand the counters to another launch."""
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
struct Late {                                // a work-group's stores, done when it waits or when its launch ends
    mutable std::vector<int *> pending;
    int add(int *p) const { return (*p)++; }
    void clear(int *p) const { pending.push_back(p); }
    void wait() const { for (int *p : pending) *p = 0; pending.clear(); }
};
int main()
{
    std::mt19937 rng(1);
    for (int groups = 1; groups <= 70; ++groups)
        for (int round = 0; round < 20; ++round) {
            std::vector<int> order(groups);
            for (int i = 0; i < groups; ++i) order[i] = i;
            std::shuffle(order.begin(), order.end(), rng);
            std::vector<Late> of(groups);
            int told = 0;
            for (int i = 0; i < groups; ++i)
                if (arrive(of[i], counters, groups, order[i])) {
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
