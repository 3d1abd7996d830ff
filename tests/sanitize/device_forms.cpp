// Host-only driver of tests/test_device_forms.py, run under AddressSanitizer + UndefinedBehaviorSanitizer and under
// ThreadSanitizer: the two device forms of weights whose sizes cut units, tiles and segments, read back.  Exit status 0 =
// the first form holds the layout's steps exactly, and the second the weight: every value once, at the row of its k.
#include <cstdint>
#include <cstdio>
#include <vector>

#include "spmm_internal.h"
#include "team.h"

using namespace spmm;

static uint32_t rng_state = 2463534242u;
static uint32_t rnd() { rng_state = rng_state * 1664525u + 1013904223u; return rng_state >> 8; }

static int first_form(const Bsr& b, const HostLayout& from_forms, const DeviceForms& f)
{
    HostLayout hl;
    layout_from_bsr(b, SEGMENT_ROWS, hl);
    std::vector<uint8_t> vals(hl.vals.size());
    std::vector<uint32_t> idx(hl.idx.size());
    if (hl.nsteps != from_forms.nsteps || hl.seg_ptr != from_forms.seg_ptr || hl.rowsum != from_forms.rowsum) return 1;
    export_steps(from_forms, f, vals.data(), idx.data());
    return vals == hl.vals && idx == hl.idx ? 0 : 2;
}

static int wide_form(const std::vector<int8_t>& W, const Bsr& b, const DeviceForms& f)
{
    const int64_t N = b.N, K = b.K, nt = ((N + TILE_ROWS - 1) / TILE_ROWS + 1) / 2, ns = (K + SEGMENT_ROWS - 1) / SEGMENT_ROWS;
    const uint8_t* const form = f.wide_bytes();
    const int32_t* const rowsum = (const int32_t*)form;
    const int32_t* const bounds = (const int32_t*)(form + wide_bounds_offset(nt));
    const uint8_t* const rec = form + wide_records_offset(nt, ns);
    const int64_t records = (f.wide_size - wide_records_offset(nt, ns)) / WIDE_RECORD_BYTES;
    std::vector<int8_t> back((size_t)(nt * WIDE_ROWS * K), 0);
    int64_t steps = 0;
    for (int64_t t = 0; t < nt; ++t)
        for (int64_t s = 0; s < ns; ++s) {
            const int32_t first = bounds[t * (ns + 1) + s], past = bounds[t * (ns + 1) + s + 1];
            if (first < 0 || past < first || past > records || past - first > f.wide_max_steps) return 10;
            if (s == 0 && f.wide_tile_steps && first != t * f.wide_tile_steps) return 11;
            steps += past - first;
            for (int32_t i = first; i < past; ++i) {
                const uint8_t* const r = rec + (int64_t)i * WIDE_RECORD_BYTES;
                const uint32_t* const sel = (const uint32_t*)(r + WIDE_VAL_BYTES);
                const uint16_t* const rows = (const uint16_t*)(r + WIDE_VAL_BYTES);
                for (int lane = 0; lane < 64; ++lane)
                    for (int e = 0; e < 16; ++e) {
                        const int z = 32 * (e >> 3) + 16 * (lane >> 5) + 4 * ((e & 7) >> 1) + (int)(sel[2 * lane] >> (2 * e) & 3);
                        const int at = 32 * (z >> 5) + 2 * (z & 7) + (z >> 4 & 1), half = 2 + (z >> 3 & 1);
                        const int row = rows[4 * at + half];
                        if (row != rows[4 * (at + 16) + half] || row % 32 || row / 32 >= SEGMENT_ROWS) return 12;
                        const int8_t v = (int8_t)r[lane * 16 + e];
                        const int64_t k = s * SEGMENT_ROWS + row / 32;
                        if (k >= K) return 13;
                        if (!v) continue;
                        int8_t& to = back[(size_t)((t * WIDE_ROWS + (lane & 31)) * K + k)];
                        if (to) return 14;
                        to = v;
                    }
            }
        }
    if (steps != f.wide_nsteps) return 15;
    for (int64_t n = 0; n < nt * WIDE_ROWS; ++n) {
        int32_t sum = 0;
        for (int64_t k = 0; k < K; ++k) {
            const int8_t w = n < N ? W[(size_t)(n * K + k)] : 0;
            if (w != back[(size_t)(n * K + k)]) return 16;
            sum += w;
        }
        if (sum != rowsum[n]) return 17;
    }
    return 0;
}

int main()
{
    const int64_t shapes[][2] = {{1, 1}, {3, 5}, {17, 64}, {33, 513}, {96, 1025}, {250, 777}, {300, 2600}, {40, 9000}};
    const int densities[] = {0, 1, 10, 25, 40, 70, 100};
    int forms = 0, without = 0;
    for (const spmm_block_t block : {SPMM_BLOCK_N4K1, SPMM_BLOCK_N1K4})
        for (const auto& shape : shapes)
            for (const int density : densities) {
                const int64_t N = shape[0], K = shape[1];
                const bool n4 = block == SPMM_BLOCK_N4K1;
                std::vector<int8_t> W((size_t)(N * K), 0);
                for (int64_t u = 0; u < (n4 ? (N + 3) / 4 : N); ++u)
                    for (int64_t c = 0; c < (n4 ? K : (K + 3) / 4); ++c) {
                        if ((int)(rnd() % 100) >= density) continue;
                        for (int j = 0; j < 4; ++j) {
                            const int64_t n = n4 ? 4 * u + j : u, k = n4 ? c : 4 * c + j;
                            if (n < N && k < K) W[(size_t)(n * K + k)] = (int8_t)((int)(rnd() % 256) - 128);
                        }
                    }
                Team team;
                Bsr b;
                bsr_from_dense(W.data(), N, K, K, block, b, team);
                HostLayout hl;
                DeviceForms f;
                int called = 0;
                forms_from_bsr(b, hl, f, team, [&] { ++called; });
                int rc = called == 1 ? first_form(b, hl, f) : 3;
                if (!rc && f.wide_size) rc = wide_form(W, b, f);
                (f.wide_size ? forms : without)++;
                // (8 steps have room for two of every four k of a row: not for all 512 of a segment, and for a quarter of them
                // wherever the packer's exchanges reach)
                if (!rc && n4 && K > SEGMENT_ROWS && density == 100 && f.wide_size) rc = 20;
                if (!rc && n4 && density <= 25 && !f.wide_size) rc = 21;
                if (rc) {
                    std::printf("%ld x %ld, %d %%, %s: %d\n", (long)N, (long)K, density, n4 ? "4x1" : "1x4", rc);
                    return 1;
                }
            }
    std::printf("ok %d %d\n", forms, without);
    return 0;
}
