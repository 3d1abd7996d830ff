// Of tests/test_device_pack.py: the forms that the device makes, read back, against the host's, byte for byte.  Two builds of it: a
// driver with the kernels on the CPU (see include/hip/hip_runtime.h), usage: device_pack N K percent n4k1|n1k4 jitter; and a shared
// object beside the product library, which is called where there is a GPU.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "spmm_internal.h"
#include "team.h"

using namespace spmm;

// 0: the same bytes
extern "C" int device_pack_bytes(int64_t N, int64_t K, int percent, int n4, int jitter, int64_t* wide_size, int64_t* nsteps)
{
    uint32_t seed = 12345u + (uint32_t)(N * 31 + K);
    auto random = [&](uint32_t n) { return (uint32_t)((uint64_t)(seed = seed * 1664525u + 1013904223u) * n >> 32); };
    std::vector<int8_t> W((size_t)(N * K), 0);
    for (int64_t n = 0; n < N; n += n4 ? 4 : 1) {
        const uint32_t keep = (uint32_t)std::max(0, 100 * percent + (jitter ? (int)random(200 * jitter + 1) - 100 * jitter : 0));
        for (int64_t k = 0; k < K; k += n4 ? 1 : 4)
            if (random(10000) < keep)
                for (int64_t j = 0; j < 4; ++j) {
                    const int64_t row = n + (n4 ? j : 0), at = k + (n4 ? 0 : j);
                    if (row < N && at < K) W[(size_t)(row * K + at)] = (int8_t)random(256);      // (0 among them)
                }
    }
    const spmm_block_t block = n4 ? SPMM_BLOCK_N4K1 : SPMM_BLOCK_N1K4;
    Bsr b;
    HostLayout hl, hl2;
    DeviceForms f, f2;
    Team team;
    bsr_from_dense(W.data(), N, K, K, block, b, team);
    forms_from_bsr(b, hl, f, team, [] {});
    uint8_t* weight = nullptr;
    DevicePack pack;
    if (!pack.reserve(N, K, block)) return 3;
    pack.begin(W.data());
    if (pack.finish(hl2, f2, &weight)) return 4;
    if (hl.nsteps != hl2.nsteps || hl.seg_ptr != hl2.seg_ptr || hl.rowsum != hl2.rowsum || hl.max_steps_per_tile != hl2.max_steps_per_tile ||
        hl.max_steps_per_segment != hl2.max_steps_per_segment || hl.nseg != hl2.nseg || hl.ntiles != hl2.ntiles || hl.kc != hl2.kc) return 5;
    if (f.size != f2.size || f.wide_size != f2.wide_size || f.tile_steps != f2.tile_steps || f.wide_tile_steps != f2.wide_tile_steps ||
        f.wide_max_steps != f2.wide_max_steps || f.wide_nsteps != f2.wide_nsteps) return 6;
    std::vector<uint8_t> back((size_t)(f2.size + f2.wide_size));
    const hipError_t e = hipMemcpy(back.data(), weight, back.size(), hipMemcpyDeviceToHost);
    (void)hipFree(weight);
    if (e != hipSuccess) return 9;
    if (std::memcmp(back.data(), f.bytes.get(), (size_t)f.size)) return 7;
    if (f.wide_size && std::memcmp(back.data() + f2.size, f.wide_bytes(), (size_t)f.wide_size)) return 8;
    *wide_size = f.wide_size;
    *nsteps = hl.nsteps;
    return 0;
}

int main(int argc, char** argv)
{
    if (argc != 6) return 2;
    int64_t wide_size = 0, nsteps = 0;
    const int rc = device_pack_bytes(atoll(argv[1]), atoll(argv[2]), atoi(argv[3]), argv[4][1] == '4', atoi(argv[5]), &wide_size, &nsteps);
    if (!rc) std::printf("ok %lld %lld\n", (long long)wide_size, (long long)nsteps);
    return rc;
}
