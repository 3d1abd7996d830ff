"""The host time of packing onto the device, relative to a weight of the same size on the same machine."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CXX = shutil.which("clang++") or "/opt/rocm/llvm/bin/clang++"
pytestmark = pytest.mark.skipif(not os.path.exists(CXX), reason="no clang++")


def run(tmp_path, source):
    src, exe, csrc = tmp_path / "driver.cpp", str(tmp_path / "driver"), os.path.join(ROOT, "paper_2306_16601_amd", "csrc")
    src.write_text(source)
    subprocess.run([CXX, "-O2", "-std=c++17", "-pthread", "-I", os.path.join(ROOT, "include"), "-I", csrc, os.path.join(csrc, "pack.cpp"), str(src),
                    "-o", exe], check=True)
    return subprocess.run([exe], capture_output=True, text=True, timeout=300, check=True).stdout


FORMS = r"""
#include <chrono>
#include <cstdint>
#include <cstdio>
#include <vector>
#include "spmm_internal.h"
#include "team.h"
using namespace spmm;

int main()
{
    const int64_t N = 256, K = 256;
    const int percent[] = {10, 30};
    Bsr weight[2];
    uint32_t seed = 777;
    for (int i = 0; i < 2; ++i) {
        std::vector<int8_t> W((size_t)(N * K), 0);
        for (int64_t block = 0; block < N * K / 4; ++block) {
            seed = seed * 1664525u + 1013904223u;
            if ((int)((seed >> 8) % 100) < percent[i])
                for (int64_t j = 0; j < 4; ++j) W[(size_t)(4 * block + j)] = (int8_t)(1 + (seed >> 9) % 127);
        }
        bsr_from_dense(W.data(), N, K, K, SPMM_BLOCK_N1K4, weight[i]);
    }
    double best[2] = {1e9, 1e9};
    for (int round = 0; round < 100; ++round)
        for (int i = 0; i < 2; ++i) {
            const auto t = std::chrono::steady_clock::now();
            Team team;
            HostLayout hl;
            DeviceForms f;
            forms_from_bsr(weight[i], hl, f, team, [] {});
            const double us = std::chrono::duration<double>(std::chrono::steady_clock::now() - t).count() * 1e6;
            if (us < best[i]) best[i] = us;
            if (i == 1 && f.wide_max_steps <= 4) return 1;      // (it needs more steps than its lists ask for)
        }
    std::printf("%f %f\n", best[0], best[1]);
}
"""


def test_lists_that_need_exchanges_and_more_steps_cost_little_more(tmp_path):
    """1x4 blocks at 70 %, where a quad's two of four are short and every tile needs a step more than its list asks for, against
    90 %: three times the blocks.  Both forms take 2.3 times as long (7 times, when every left-over k was tried slot by slot,
    and every tile arranged a second time)."""
    sparse, dense = (float(v) for v in run(tmp_path, FORMS).split())
    assert dense < 4 * sparse, (dense, sparse)


THREADS = r"""
#include <chrono>
#include <cstdio>
#include <filesystem>
#include <iterator>
#include <set>
#include "team.h"
using namespace spmm;

int main()
{
    auto threads = [] { return std::distance(std::filesystem::directory_iterator("/proc/self/task"), std::filesystem::directory_iterator()); };
    for (const int pieces : {1, 2, 3, 20}) {
        std::atomic<long> most{0};
        std::atomic<int> done{0};
        {
            Team team;
            for (int pass = 0; pass < 3; ++pass)
                team.run(pieces, 1, [&](int64_t, int64_t) {
                    std::this_thread::sleep_for(std::chrono::milliseconds(20));     // (time for any other thread to start)
                    const long now = threads();
                    for (long seen = most; seen < now && !most.compare_exchange_weak(seen, now);) {}
                    ++done;
                });
            team.finish(100, 1, [&](int64_t, int64_t) { ++done; });
        }
        if (done != 3 * pieces + 100) return 1;
        std::printf("%d %ld\n", pieces, (long)most);
    }
}
"""


def test_a_weight_of_two_pieces_starts_one_thread(tmp_path):
    """(The threads are started by each other, 15 to 30 us each: for small weights that was half of the time.)"""
    for line in run(tmp_path, THREADS).splitlines():
        pieces, threads = (int(v) for v in line.split())
        assert 1 <= threads <= min(pieces, 8), (pieces, threads)
