"""The work list of the region passes (csrc/worklist.hpp) on the host: the header
is compiled with g++ against stand-ins for the wavefront intrinsics, 256 threads
run it as a workgroup, and each of the four wavefronts is given its own reading
of the case's error bits, as it happens when the lattice kernel on the other
stream flags the case in between.  Every cell handed out must be a marked one of
the region, each at most once and all of those of the wavefronts that read no
error, whatever the list's memory held before."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2408_15115_amd", "csrc")

HARNESS = r"""
#include <atomic>
#include <barrier>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <random>
#include <thread>
#include <vector>
#define __device__
static thread_local struct { unsigned x; } threadIdx;
static std::unique_ptr<std::barrier<>> workgroup, wave[4];
static std::atomic<unsigned long long> votes[4];
static unsigned long long __ballot(bool v)
{
    const int w = threadIdx.x >> 6;
    if (v) votes[w] |= 1ull << (threadIdx.x & 63);
    wave[w]->arrive_and_wait();
    const unsigned long long m = votes[w];
    wave[w]->arrive_and_wait();
    if ((threadIdx.x & 63) == 0) votes[w] = 0;
    wave[w]->arrive_and_wait();
    return m;
}
static int __popcll(unsigned long long v) { return __builtin_popcountll(v); }
static void __syncthreads() { workgroup->arrive_and_wait(); }
#include "worklist.hpp"

// early: the wavefronts that read an error leave before the list
static int faults(int first, int count, const int err[4], bool early, std::mt19937 &rng)
{
    std::vector<unsigned char> marks(count);
    for (auto &m : marks) m = rng() % 3 == 0;
    turret::ScanList list;   // what an earlier workgroup left
    std::memset(&list, 0, sizeof list);
    for (auto &n : list.n) n = 20 + rng() % 20;
    for (auto &a : list.at) a = (unsigned char)rng();
    workgroup = std::make_unique<std::barrier<>>(256);
    for (auto &w : wave) w = std::make_unique<std::barrier<>>(64);
    std::vector<int> got(256, -1);
    std::vector<std::thread> threads;
    for (unsigned t = 0; t < 256; t++)
        threads.emplace_back([&, t] {
            threadIdx.x = t;
            const int e = err[t >> 6];
            if (early && e != 0) {
                workgroup->arrive_and_drop();
                return;
            }
            got[t] = turret::scan_cells(list, first, count, e, [&](int i) { return marks.at(i); });
        });
    for (auto &t : threads) t.join();
    int bad = 0;
    std::vector<int> times(count, 0);
    for (int q : got) {
        if (q == -1) continue;
        if (q < first || q >= count || !marks[q]) bad++;
        else if (times[q]++) bad++;
    }
    for (int i = first; i < std::min(first + 256, count); i++)
        if (err[(i - first) >> 6] == 0 && marks[i] && times[i] != 1) bad++;
    return bad;
}

int main(int, char **argv)
{
    std::mt19937 rng(5);
    const bool early = std::atoi(argv[1]) != 0;
    int bad = 0;
    for (int mask = 0; mask < 16; mask++) {
        const int err[4] = {mask & 1 ? 4 : 0, mask & 2 ? 4 : 0, mask & 4 ? 4 : 0, mask & 8 ? 4 : 0};
        bad += faults(0, 4096, err, early, rng);          // a whole block
        bad += faults(2816, 2816 + 65, err, early, rng);  // the last block of a region, ragged
    }
    std::printf("%d\n", bad);
}
"""


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    d = tmp_path_factory.mktemp("worklist")
    (d / "harness.cpp").write_text(HARNESS)
    exe = str(d / "harness")
    subprocess.check_call(["g++", "-std=c++20", "-O1", "-g", "-pthread", "-Wall", "-I", CSRC, str(d / "harness.cpp"), "-o", exe])
    return lambda early: int(subprocess.run([exe, str(early)], capture_output=True, text=True, check=True, timeout=120).stdout)


def test_wavefronts_that_disagree_on_the_error_bits_share_a_sound_list(harness):
    assert harness(0) == 0


def test_the_harness_sees_wavefronts_that_leave_early(harness):
    assert harness(1) > 0
