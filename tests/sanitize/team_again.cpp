// Host-only driver of tests/test_team.py: a weight's canonical form made with something beside its passes, as packing on the device
// makes it, and then the device forms with the same threads, as where the device has no memory for them.  Exit status 0 = the passes
// after that are shared again, with the same results.
#include <chrono>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <set>
#include <stdexcept>
#include <thread>
#include <vector>

#include "spmm_internal.h"
#include "team.h"

using namespace spmm;

// a pass of 64 pieces of a millisecond is not the calling thread's alone
static bool shared(Team& team)
{
    std::mutex mutex;
    std::set<std::thread::id> seen;
    team.run(64, 1, [&](int64_t, int64_t) {
        std::this_thread::sleep_for(std::chrono::milliseconds(1));
        const std::lock_guard<std::mutex> lock(mutex);
        seen.insert(std::this_thread::get_id());
    });
    return seen.size() > 1;
}

int main()
{
    const int64_t N = 2048, K = 1024;
    std::vector<int8_t> W((size_t)(N * K), 0);
    for (int64_t i = 0; i < N * K; i += 4) W[(size_t)i] = (int8_t)(i % 251 - 120);
    Team first;
    const bool can = shared(first);
    for (int round = 0; round < 20; ++round) {
        Team team;
        Bsr b, again;
        int own = 0;
        const Beside beside = {[&] { ++own; }, [&] { ++own; }};
        bsr_from_dense(W.data(), N, K, K, SPMM_BLOCK_N4K1, b, team, &beside);
        if (own != 2) return 1;
        if (round % 2) {
            HostLayout hl, alone;
            DeviceForms f, g;
            forms_from_bsr(b, hl, f, team, [] {});
            Team other;
            forms_from_bsr(b, alone, g, other, [] {});
            if (hl.seg_ptr != alone.seg_ptr || hl.rowsum != alone.rowsum || f.size != g.size || std::memcmp(f.bytes.get(), g.bytes.get(), (size_t)f.size)) return 2;
        }
        if (shared(team) != can) return 3;
        bsr_from_dense(W.data(), N, K, K, SPMM_BLOCK_N4K1, again, team, &beside);
        if (again.index != b.index || again.vals != b.vals) return 4;
        bool failed = false;
        try {
            team.finish(64, 1, [](int64_t i, int64_t) { if (i == 40) throw std::runtime_error("piece"); });
        } catch (const std::runtime_error&) {
            failed = true;
        }
        if (!failed || shared(team) != can) return 5;
    }
    std::printf("ok %d\n", can);
    return 0;
}
