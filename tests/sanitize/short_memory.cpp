// Host-only driver of tests/test_short_memory.py, under AddressSanitizer + UndefinedBehaviorSanitizer: both device forms of a
// weight, with every host allocation from the second form's own buffer on failing in turn.  Exit status 0 = no exception,
// no second form, and the first one the same as ever.
#include <atomic>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>

#include "spmm_internal.h"
#include "team.h"

using namespace spmm;

static std::atomic<size_t> failing_size{0};
static std::atomic<int> failed{0};
void* operator new[](size_t n)
{
    if (failing_size && n == failing_size) {
        ++failed;
        throw std::bad_alloc();
    }
    void* const p = std::malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete[](void* p) noexcept { std::free(p); }
void operator delete[](void* p, size_t) noexcept { std::free(p); }

int main()
{
    struct Weight { int64_t N, K; spmm_block_t block; int percent; };
    uint32_t seed = 12345;
    // (the last needs more steps than its lists ask for: its second form is packed twice, into buffers of two sizes)
    for (const Weight& w : {Weight{800, 1100, SPMM_BLOCK_N4K1, 20}, Weight{800, 1100, SPMM_BLOCK_N1K4, 18}, Weight{1600, 300, SPMM_BLOCK_N1K4, 30}}) {
        const int64_t N = w.N, K = w.K;
        const spmm_block_t block = w.block;
        const bool n4 = block == SPMM_BLOCK_N4K1;
        std::vector<int8_t> W((size_t)(N * K), 0);
        for (int64_t i = 0; i < N * K / 4; ++i) {
            seed = seed * 1664525u + 1013904223u;
            if ((int)((seed >> 8) % 100) < w.percent)
                for (int64_t j = 0; j < 4; ++j) W[(size_t)(n4 ? (i / K * 4 + j) * K + i % K : 4 * i + j)] = (int8_t)(1 + (seed >> 9) % 100);
        }
        auto pack = [&](HostLayout& hl, DeviceForms& f) {
            Team team;
            Bsr b;
            bsr_from_dense(W.data(), N, K, K, block, b, team);
            forms_from_bsr(b, hl, f, team, [] {});
        };
        HostLayout hl;
        DeviceForms whole;
        pack(hl, whole);
        if (whole.together || !whole.wide_size) return 2;
        if (K == 300 && whole.wide_max_steps <= 5) return 6;
        // the second form's buffer; and the scratch of the threads that fill it (other sizes than any of the first form's)
        const int64_t units = n4 ? WIDE_ROWS / 4 : WIDE_ROWS;
        const size_t sizes[] = {(size_t)whole.wide_size, (size_t)(2 * hl.nseg * WIDE_MAX_STEPS * units * 4)};
        for (const size_t size : sizes) {
            HostLayout hl2;
            DeviceForms f;
            failed = 0;
            failing_size = size;
            try {
                pack(hl2, f);
            } catch (...) {
                std::printf("%ld x %ld: size %zu: an exception\n", (long)N, (long)K, size);
                return 3;
            }
            failing_size = 0;
            if (!failed || f.wide_size || f.wide_max_steps || f.wide_nsteps || f.wide) return 4;
            if (f.size != whole.size || std::memcmp(f.bytes.get(), whole.bytes.get(), (size_t)f.size) != 0) return 5;
        }
    }
    std::printf("ok\n");
    return 0;
}
