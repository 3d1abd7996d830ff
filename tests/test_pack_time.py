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


CANONICAL = r"""
#include <chrono>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <vector>
#include "spmm_internal.h"
#include "team.h"
using namespace spmm;

// the blocks of a weight in one pass, to memory that is there
static int64_t one_pass(const int8_t* W, int64_t N, int64_t K, int32_t* index, int8_t* vals)
{
    int64_t n = 0;
    for (int64_t row = 0; row < N; ++row)
        for (int64_t c = 0; c * 4 < K; ++c) {
            uint32_t v = 0;
            std::memcpy(&v, W + row * K + 4 * c, (size_t)(K - 4 * c < 4 ? K - 4 * c : 4));
            if (v) {
                index[n] = (int32_t)c;
                std::memcpy(vals + 4 * n++, &v, 4);
            }
        }
    return n;
}

int main()
{
    const int64_t N = 256, K = 256;
    std::vector<int8_t> W((size_t)(N * K), 0);
    uint32_t seed = 777;
    for (int64_t block = 0; block < N * K / 4; ++block) {
        seed = seed * 1664525u + 1013904223u;
        if ((seed >> 8) % 100 < 20)
            for (int64_t j = 0; j < 4; ++j) W[(size_t)(4 * block + j)] = (int8_t)(1 + (seed >> 9) % 127);
    }
    std::vector<int32_t> index((size_t)(N * K / 4));
    std::vector<int8_t> vals((size_t)(N * K));
    double best[2] = {1e9, 1e9};
    for (int round = 0; round < 200; ++round)
        for (int i = 0; i < 2; ++i) {
            const auto t = std::chrono::steady_clock::now();
            int64_t n = 0;
            if (i) {
                Team team;
                Bsr b;
                bsr_from_dense(W.data(), N, K, K, SPMM_BLOCK_N1K4, b, team);
                n = (int64_t)b.index.size();
            } else {
                n = one_pass(W.data(), N, K, index.data(), vals.data());
            }
            const double us = std::chrono::duration<double>(std::chrono::steady_clock::now() - t).count() * 1e6;
            if (us < best[i]) best[i] = us;
            if (n < N * K / 4 / 6) return 1;
        }
    std::printf("%f %f\n", best[0], best[1]);
}
"""


def test_1x4_blocks_counted_and_listed_cost_little_more_than_listed(tmp_path):
    """The canonical form in its two passes takes 1.3 times as long as one pass over the weight that lists the same blocks (9 times,
    when the length of the last one was in question at every block, in both passes)."""
    once, counted = (float(v) for v in run(tmp_path, CANONICAL).split())
    assert counted < 3 * once, (counted, once)
