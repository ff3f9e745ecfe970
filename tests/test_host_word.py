"""The pinned words that compressing calls read their counts from (csrc/host_word.h), on the CPU with stand-ins for the runtime: a word
that a kernel may still write is not handed to another call, whichever way the first one ended."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

PROGRAM = r"""
#include "host_word.h"
#include <cstdio>
#include <cstdlib>
#include <set>
static int room[64 * 16], synced = hipSuccess, copies = 0;
static bool refuse = REFUSE;
hipError_t hipHostMalloc(void **p, size_t, unsigned) { *p = room; return refuse ? hipErrorOutOfMemory : hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return (hipError_t)synced; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t, hipMemcpyKind, hipStream_t) { ++copies; *(int *)d = *(const int *)s; return hipSuccess; }
using fscnn::HostWord;
#define CHECK(c) do { if (!(c)) { std::printf("line %d: " #c "\n", __LINE__); std::exit(1); } } while (0)
int main()
{
    int out = 0, on_device = 7;
    if (refuse) {
        HostWord w;
        CHECK(!w.hand_out() && w.wait(&on_device, nullptr, &out) == hipSuccess && out == 7 && copies == 1);
        return 0;
    }
    std::set<int *> lost, seen;
    int *p = nullptr;
    { HostWord w; p = w.hand_out(); *p = 41; CHECK(w.wait(&on_device, nullptr, &out) == hipSuccess && out == 41); }
    { HostWord w; CHECK(w.hand_out() == p); lost.insert(p); }                         // an error before wait()
    { HostWord w; p = w.hand_out(); CHECK(!lost.count(p)); lost.insert(p); synced = hipErrorUnknown; CHECK(w.wait(&on_device, nullptr, &out) != hipSuccess); synced = hipSuccess; }
    { HostWord w; (void)w; }                                                          // an error before any launch
    { HostWord w[64]; for (auto &q : w) { int *r = q.hand_out(); if (r) CHECK(!lost.count(r) && seen.insert(r).second); CHECK(q.wait(&on_device, nullptr, &out) == hipSuccess); } }
    CHECK(seen.size() == 62 && copies == 2);
    return 0;
}
"""


@pytest.mark.parametrize("refuse", [False, True])
def test_words_that_may_be_written_are_not_reused(tmp_path, refuse):
    src, exe = tmp_path / "words.cpp", tmp_path / "words"
    src.write_text(PROGRAM.replace("REFUSE", "true" if refuse else "false"))
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
                    "-I", os.path.join(ROOT, "paper_2212_08815_amd", "csrc"), str(src), "-o", str(exe), "-lpthread"], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


UNWRITTEN = PROGRAM[:PROGRAM.index("int main()")] + r"""
int main()
{
    int out = 0, on_device = 7, *p = nullptr;
    { HostWord w; p = w.hand_out(); CHECK(w.wait(&on_device, nullptr, &out) == hipSuccess && out < 0); }     // the stream ended, nothing was written
    { HostWord w; CHECK(w.hand_out() != p); *w.hand_out() = 3; CHECK(w.wait(&on_device, nullptr, &out) == hipSuccess && out == 3); }
    return 0;
}
"""


def test_a_word_that_nothing_wrote_is_no_number_and_not_reused(tmp_path):
    src, exe = tmp_path / "unwritten.cpp", tmp_path / "unwritten"
    src.write_text(UNWRITTEN.replace("REFUSE", "false"))
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
                    "-I", os.path.join(ROOT, "paper_2212_08815_amd", "csrc"), str(src), "-o", str(exe), "-lpthread"], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


SECOND = PROGRAM[:PROGRAM.index("int main()")] + r"""
int main()
{
    int out = 0, few = 0, on_device[2] = {7, 3};
    HostWord w;
    if (int *p = w.hand_out()) { p[0] = 41; p[1] = 5; }
    CHECK(w.wait(on_device, nullptr, &out, &few) == hipSuccess && out == (refuse ? 7 : 41) && few == (refuse ? 3 : 5) && copies == (refuse ? 2 : 0));
    return 0;
}
"""


@pytest.mark.parametrize("refuse", [False, True])
def test_the_number_behind_the_word(tmp_path, refuse):
    src, exe = tmp_path / "second.cpp", tmp_path / "second"
    src.write_text(SECOND.replace("REFUSE", "true" if refuse else "false"))
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
                    "-I", os.path.join(ROOT, "paper_2212_08815_amd", "csrc"), str(src), "-o", str(exe), "-lpthread"], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
