"""The workgroup sums of output counts (csrc/group_scan.hpp), the device code
itself compiled for the host: a thread per lane, shuffles and barriers through
shared memory.  Rows of 2^25 entries and more, whose sum over one workgroup
leaves 32 bits, cannot be had on a GPU in a test's time."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = r"""
#include <barrier>
#include <cstdint>
#include <cstdio>
#include <thread>
#include <vector>
#define __device__
#define __forceinline__ inline
struct Index { unsigned x; };
static thread_local Index threadIdx;
static std::barrier<> *bar;
static int64_t slot[128];
static void __syncthreads() { bar->arrive_and_wait(); }
template <typename T> static T __shfl_up(T v, int off) {  // over waves of 64
    const int t = threadIdx.x;
    slot[t] = v;
    bar->arrive_and_wait();
    const T u = static_cast<T>(slot[t % 64 >= off ? t - off : t]);
    bar->arrive_and_wait();
    return u;
}
#include "group_scan.hpp"
template <int T> static void run(const std::vector<int32_t> &count) {
    std::barrier<> b(T);
    bar = &b;
    int64_t s_wave[T / 64], upto[T], all[T];
    std::vector<std::thread> lanes;
    for (int t = 0; t < T; ++t)
        lanes.emplace_back([&, t] {
            threadIdx.x = t;
            upto[t] = spl::group_inclusive<T>(count[t], s_wave, &all[t]);
        });
    for (auto &l : lanes) l.join();
    for (int t = 0; t < T; ++t)
        std::printf("%lld %lld\n", static_cast<long long>(upto[t]), static_cast<long long>(all[t]));
}
int main(int argc, char **argv) {
    std::vector<int32_t> count;
    long long c;
    while (std::scanf("%lld", &c) == 1) count.push_back(static_cast<int32_t>(c));
    if (count.size() == 64) run<64>(count);
    else if (count.size() == 128) run<128>(count);
    else return 1;
}
"""


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    d = tmp_path_factory.mktemp("group_scan")
    src, exe = d / "t.cpp", d / "t"
    src.write_text(HARNESS)
    subprocess.run(["g++", "-std=c++20", "-O1", "-pthread", "-Wno-unknown-pragmas", "-I",
                    os.path.join(ROOT, "paper_2207_13901_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    return exe


@pytest.mark.parametrize("lanes", (64, 128))
@pytest.mark.parametrize("count", (7, 2 ** 25 + 1, 75_000_000, 2 ** 31 - 1))
def test_sums_over_a_workgroup(harness, lanes, count):
    counts = [count - (k % 3) for k in range(lanes)]
    out = subprocess.run([str(harness)], input=" ".join(map(str, counts)), text=True,
                         capture_output=True, check=True, timeout=60).stdout.split("\n")
    upto = 0
    for k in range(lanes):
        upto += counts[k]
        assert out[k].split() == [str(upto), str(sum(counts))], k
