// Packing of large weights on the device: both device forms (spmm_internal.h) from the dense weight, byte for byte what
// forms_from_bsr in pack.cpp makes of it.
//
// What bounds a pack is the host: its passes over the weight and the forms, and the pages of the buffers between them.  The dense
// weight is on the device in a fifth of the time in which 8 threads make the forms of it, and a workgroup per (32 rows, 512 k)
// needs nothing else.  So the canonical form is made by the host's threads while the weight is on its way and its lists are dealt
// to slots (spmm_pack_lists); the numbers of steps come back, which say where every record goes, and they are written there
// (spmm_pack_records).  1024x4096 at 80 %: the pack 800 to 870 -> 350 us, of which the copy 135, the lists 45 (one wave's chain of 450
// slots, at 0.1 us each), the records 17; packed, unpacked and released 1.22 to 1.36 -> 0.58 to 0.63 ms (machines differ);
// 4096x4096 at 70 % 3.6 -> 0.98 ms, 1x4 blocks of 4096x1024 at 90 % 1.37 -> 0.39.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

#include "spmm_internal.h"

namespace spmm {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
struct __attribute__((packed)) v4i_anywhere { v4i v; };

constexpr int THREADS = 256;
constexpr int PITCH = SEGMENT_ROWS + 16;    // of a row in LDS: rows start 4 banks apart
constexpr int MAX_QUADS = WIDE_MAX_STEPS * STEP_K / 4;

struct PackArgs {
    const int8_t* W;            // [N][K]
    int32_t* info;              // steps of every (row tile, segment), of every (wide tile, segment) (-1: too many), and the sums of
                                // 32 rows of every (wide tile, segment)
    int16_t *slots, *wide_slots;        // [row tile, or wide tile][segment][512]: the k of a slot, negative: padding (narrow: ~row)
    const uint8_t* heads;       // what stands in front of the records of the first form, and of the wide one
    uint8_t *weight, *wide;     // the forms (wide: or null)
    int64_t head_dwords, wide_head_dwords;
    int64_t N;
    int K, nseg, ntiles, tile_steps, wide_tile_steps;
    bool n4;
};

// what lanes of a wave read after this, other lanes of it wrote before
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ int set_bits(const uint32_t v) { return __builtin_popcount(v); }
__device__ __forceinline__ int set_bits64(const uint64_t v) { return __builtin_popcountll(v); }

// 32 rows x 512 k of the weight, zero past its ends
__device__ __forceinline__ void load_tile(const PackArgs& a, const int64_t t, const int seg, uint8_t* const tile)
{
#pragma unroll
    for (int i = 0; i < WIDE_ROWS * (SEGMENT_ROWS / 16) / THREADS; ++i) {
        const int p = (int)threadIdx.x + i * THREADS, row = p / (SEGMENT_ROWS / 16), col = p % (SEGMENT_ROWS / 16) * 16;
        const int64_t n = t * WIDE_ROWS + row;
        const int k = seg * SEGMENT_ROWS + col;
        v4i v = {0, 0, 0, 0};
        if (n < a.N) {
            const int8_t* const from = a.W + n * a.K + k;
            if (k + 16 <= a.K) {
                v = ((const v4i_anywhere*)from)->v;
            } else {
                for (int j = 0; j < 16; ++j)
                    if (k + j < a.K) v[j >> 2] |= (int)((uint32_t)(uint8_t)from[j] << (8 * (j & 3)));
            }
        }
        *(v4i*)(tile + row * PITCH + col) = v;
    }
}

// of every k, the units that list it: bit u for block-row u, or row u of 1x4 blocks
__device__ __forceinline__ void find_masks(const bool n4, const uint8_t* const tile, uint32_t* const mask)
{
    if (threadIdx.x >= SEGMENT_ROWS / 4) return;
    const uint8_t* const at = tile + 4 * threadIdx.x;
    uint32_t m[4] = {0, 0, 0, 0};
    for (int u = 0; u < (n4 ? 8 : 32); ++u) {
        uint32_t w;
        if (n4) {
            const uint8_t* const r = at + 4 * u * PITCH;
            w = *(const uint32_t*)r | *(const uint32_t*)(r + PITCH) | *(const uint32_t*)(r + 2 * PITCH) | *(const uint32_t*)(r + 3 * PITCH);
        } else {
            w = *(const uint32_t*)(at + u * PITCH);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) m[j] |= (uint32_t)((w >> (8 * j) & 0xff) != 0) << u;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) mask[4 * threadIdx.x + j] = m[j];
}

// place of the nth set bit
__device__ __forceinline__ int nth_bit(uint32_t w, int nth)
{
    int at = 0;
#pragma unroll
    for (int s = 16; s >= 1; s >>= 1) {
        const int below = set_bits(w & ((1u << s) - 1));
        const bool up = nth >= below;
        nth -= up ? below : 0;
        w = up ? w >> s : w;
        at += up ? s : 0;
    }
    return at;
}

// arrange_for_lds_banks of pack.cpp by one wave, lane h for half-read h: returns the number of steps
__device__ __forceinline__ int deal_to_banks(const uint32_t* const mask, const uint32_t mine, const int rows, int16_t* const slots)
{
    const int lane = threadIdx.x & 63, residue = lane & 15, h = lane & 31;
    uint32_t listed = 0;        // bit i: k = 16 i + residue is
    for (int i = 0; i < SEGMENT_ROWS / 16; ++i) listed |= (uint32_t)((mask[16 * i + residue] & mine) != 0) << i;
    int rank = 0, total = 0;    // largest class first, stable
    for (int r = 0; r < 16; ++r) {
        const int n = set_bits((uint32_t)__builtin_amdgcn_readlane((int)listed, r)), own = set_bits(listed);
        rank += n > own || (n == own && r < residue);
        total += n;
    }
    const int nsteps = (total + STEP_K - 1) / STEP_K, H = 4 * nsteps;
    if (nsteps == 0) return 0;
    const uint32_t all = H == 32 ? ~0u : (1u << H) - 1;
    uint32_t low = all, present = 0;
    int load = 0;
    auto slot_of = [&](const int j) { return h / 4 * STEP_K + 16 * (2 * (h & 1) + j / 8) + 8 * (h / 2 % 2) + j % 8; };
    for (int oi = 0; oi < 16; ++oi) {
        const int r = __builtin_ctzll(__builtin_amdgcn_ballot_w64(lane < 16 && rank == oi));
        const uint32_t of_class = (uint32_t)__builtin_amdgcn_readlane((int)listed, r);
        const int n = set_bits(of_class);
        int next = 0;
        auto deal = [&](const uint32_t to, const int j) {
            const int given = min(set_bits(to), n - next), mine_is = set_bits(to & ((1u << h) - 1));
            const bool in = lane < 32 && (to >> h & 1) != 0, gets = in && mine_is < given;
            if (gets) {
                present |= 1u << r;
                slots[slot_of(j)] = (int16_t)(16 * nth_bit(of_class, next + mine_is) + r);
            }
            next += given;
            return (uint32_t)__builtin_amdgcn_ballot_w64(in && !gets);
        };
        while (next < n) {
            const uint32_t high = all & ~low, left = deal(low, load);
            if (left) {
                low = left;
            } else {
                low |= deal(high, load + 1);
                ++load;
            }
        }
    }
    if (lane < H) {
        int next = 0;
        for (int j = load + !(low >> h & 1); j < 16; ++j) {
            while (next < 16 && (present >> next & 1)) ++next;
            int row = 0;
            if (next < 16) {
                if (next < rows) row = next;
                present |= 1u << next;
            }
            slots[slot_of(j)] = (int16_t)~row;
        }
    }
    return nsteps;
}

struct WideScratch {
    int16_t cand[8][64];
    uint32_t one[MAX_QUADS], two[MAX_QUADS];       // units with a k, with two, in the quad
    uint64_t left[8];
};

// arrange_wide of pack.cpp by one wave, lane i for the candidate i of every class; -1: more than WIDE_MAX_STEPS
__device__ __forceinline__ int deal_to_quads(const uint32_t* const mask, const int units, WideScratch& f, int16_t* const slots)
{
    const int lane = threadIdx.x & 63;
    const uint64_t below = ((uint64_t)1 << lane) - 1;
    int k_of[8], n = 0;
    uint32_t users[8];
    uint64_t alive[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {           // heaviest first, stable; those that none uses are no candidates
        const int w = set_bits(mask[8 * lane + c]);
        int base = 0;
        for (int b = units; b > 0; --b) {
            const uint64_t these = __builtin_amdgcn_ballot_w64(w == b);
            if (w == b) f.cand[c][base + set_bits64(these & below)] = (int16_t)(8 * lane + c);
            base += set_bits64(these);
        }
        alive[c] = base == 64 ? ~(uint64_t)0 : ((uint64_t)1 << base) - 1;
        n += base;
        if (lane >= base) f.cand[c][lane] = 0;
    }
    wave_sync();
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        k_of[c] = f.cand[c][lane];
        users[c] = mask[k_of[c]];
    }
    int steps = (n + STEP_K - 1) / STEP_K;
    for (int q = lane; q < MAX_QUADS; q += 64) f.one[q] = f.two[q] = 0;
    wave_sync();
    for (int s = 0; s < steps; ++s) {
        int slot = -1;                      // slot `lane` of the step; lane q: quad q
        uint32_t one_of = 0, two_of = 0;
#pragma unroll
        for (int o = 0; o < 8; ++o) {
            uint32_t one = 0, two = 0;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int c = (j + o) & 7;
                if (j == 4) one = two = 0;
                const uint64_t fit = alive[c] & __builtin_amdgcn_ballot_w64((users[c] & two) == 0);
                if (fit) {
                    const int at = __builtin_ctzll(fit);
                    alive[c] &= ~(fit & (0 - fit));
                    const uint32_t m = (uint32_t)__builtin_amdgcn_readlane((int)users[c], at);
                    const int k = __builtin_amdgcn_readlane(k_of[c], at);
                    two |= one & m;
                    one |= m;
                    slot = lane == 8 * o + j ? k : slot;
                }
                if (j == 3 || j == 7) {
                    one_of = lane == 2 * o + j / 4 ? one : one_of;
                    two_of = lane == 2 * o + j / 4 ? two : two_of;
                }
            }
        }
        slots[s * STEP_K + lane] = (int16_t)slot;
        if (lane < 16) {
            f.one[16 * s + lane] = one_of;
            f.two[16 * s + lane] = two_of;
        }
    }
    uint64_t any = 0;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        any |= alive[c];
        if (lane == 0) f.left[c] = alive[c];
    }
    if (!any) return steps;
    wave_sync();
    // What is left over: into the first quad with a hole that it fits, by an exchange, or to a new step, as pack.cpp has it.
    auto hole = [&](const int q) {
        return q < 16 * steps && (slots[4 * q] < 0 || slots[4 * q + 1] < 0 || slots[4 * q + 2] < 0 || slots[4 * q + 3] < 0);
    };
    auto put = [&](const int z, const int k, const uint32_t m) {       // (by all lanes alike)
        const uint32_t one = f.one[z / 4], two = f.two[z / 4];
        wave_sync();
        if (lane == 0) {
            slots[z] = (int16_t)k;
            f.two[z / 4] = two | (one & m);
            f.one[z / 4] = one | m;
        }
        wave_sync();
    };
    auto fill = [&](const int q, const int k, const uint32_t m) {       // the first hole of quad q
        int z = 4 * q;
        while (slots[z] >= 0) ++z;
        put(z, k, m);
    };
    int exchanges = 256;
    for (int c = 0; c < 8; ++c) {
        uint64_t left = f.left[c];
        while (left) {
            const int k = __builtin_amdgcn_readfirstlane(f.cand[c][__builtin_ctzll(left)]);
            const uint32_t m = (uint32_t)__builtin_amdgcn_readfirstlane((int)mask[k]);
            const bool hole0 = hole(lane), hole1 = hole(lane + 64);
            const uint32_t two0 = f.two[lane], two1 = f.two[lane + 64];
            const uint64_t fits0 = __builtin_amdgcn_ballot_w64(hole0 && !(two0 & m)), fits1 = __builtin_amdgcn_ballot_w64(hole1 && !(two1 & m));
            bool done = (fits0 | fits1) != 0;
            if (done) {
                fill(fits0 ? __builtin_ctzll(fits0) : 64 + __builtin_ctzll(fits1), k, m);
            } else {
                uint64_t holes0 = __builtin_amdgcn_ballot_w64(hole0), holes1 = __builtin_amdgcn_ballot_w64(hole1);
                while ((holes0 | holes1) && !done && exchanges-- > 0) {
                    const int q = holes0 ? __builtin_ctzll(holes0) : 64 + __builtin_ctzll(holes1);
                    if (holes0) holes0 &= holes0 - 1;
                    else holes1 &= holes1 - 1;
                    const uint32_t two_q = f.two[q];
                    for (int s = 0; s < steps && !done; ++s) {
                        const int z = s * STEP_K + lane, there = slots[z];
                        const uint32_t u = there < 0 ? ~0u : mask[there], t = f.two[z / 4];
                        const uint64_t yes = __builtin_amdgcn_ballot_w64(!(m & t & ~u) && !(two_q & u) && z / 4 != q);
                        if (!yes) continue;
                        const int at = s * STEP_K + __builtin_ctzll(yes), r = at / 4;
                        const int other = slots[at];
                        const uint32_t of_other = mask[other], one_r = f.one[r], two_r = f.two[r];
                        wave_sync();
                        if (lane == 0) {
                            f.one[r] = (one_r & ~of_other) | (two_r & of_other);
                            f.two[r] = two_r & ~of_other;
                        }
                        wave_sync();
                        fill(q, other, of_other);
                        put(at, k, m);
                        done = true;
                    }
                }
            }
            if (!done) {
                if (steps == WIDE_MAX_STEPS) return -1;
                slots[steps * STEP_K + lane] = -1;
                ++steps;
                wave_sync();
                continue;
            }
            left &= left - 1;
        }
    }
    return steps;
}

// Workgroup (t, segment): the lists of wide tile t and of its two row tiles, dealt to slots.
__global__ void __launch_bounds__(THREADS) spmm_pack_lists(const PackArgs a)
{
    __shared__ __attribute__((aligned(16))) uint8_t tile[WIDE_ROWS * PITCH];
    __shared__ uint32_t mask[SEGMENT_ROWS];
    __shared__ int32_t sums[THREADS];
    __shared__ int16_t slots[3][SEGMENT_ROWS];
    __shared__ int32_t steps[3];
    __shared__ WideScratch wide;
    const int64_t t = blockIdx.x, nt = gridDim.x;
    const int seg = blockIdx.y, rows = min(SEGMENT_ROWS, a.K - seg * SEGMENT_ROWS), tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    load_tile(a, t, seg, tile);
    __syncthreads();
    find_masks(a.n4, tile, mask);
    int32_t sum = 0;
    for (int i = 0; i < 16; ++i) {
        const uint32_t w = *(const uint32_t*)(tile + (tid >> 3) * PITCH + (tid & 7) * 64 + 4 * i);
        sum += (int8_t)w + (int8_t)(w >> 8) + (int8_t)(w >> 16) + (int8_t)(w >> 24);
    }
    sums[tid] = sum;
    __syncthreads();
    if (wave < 3) {
        const uint32_t half = a.n4 ? 0xfu : 0xffffu;
        const int n = wave == 2 ? deal_to_quads(mask, a.n4 ? 8 : 32, wide, slots[2]) : deal_to_banks(mask, wave ? ~half : half, rows, slots[wave]);
        if ((tid & 63) == 0) steps[wave] = n;
    } else if ((tid & 63) < WIDE_ROWS) {
        const int row = tid & 63;
        int32_t all = 0;
        for (int i = 0; i < 8; ++i) all += sums[8 * row + i];
        a.info[(int64_t)a.ntiles * a.nseg + nt * a.nseg + (t * a.nseg + seg) * WIDE_ROWS + row] = all;
    }
    __syncthreads();
    for (int i = 0; i < 3; ++i) {
        const int64_t of = i == 2 ? t : 2 * t + i;
        if (i < 2 && of >= a.ntiles) continue;
        int16_t* const to = (i == 2 ? a.wide_slots : a.slots) + (of * a.nseg + seg) * SEGMENT_ROWS;
        for (int z = tid; z < steps[i] * STEP_K; z += THREADS) to[z] = slots[i][z];
        if (tid == 0) a.info[(i == 2 ? (int64_t)a.ntiles * a.nseg : 0) + of * a.nseg + seg] = steps[i];
    }
}

__device__ __forceinline__ void clear_records(uint8_t* const from, const int64_t bytes)
{
    for (int64_t i = 16 * (int64_t)threadIdx.x; i < bytes; i += 16 * THREADS) *(v4i*)(from + i) = (v4i){0, 0, 0, 0};
}

// Workgroup (t, segment): the records of its lists, and with the last segment the unused ones of the tiles.
__global__ void __launch_bounds__(THREADS) spmm_pack_records(const PackArgs a)
{
    __shared__ __attribute__((aligned(16))) uint8_t tile[WIDE_ROWS * PITCH];
    __shared__ uint32_t mask[SEGMENT_ROWS];
    __shared__ int16_t slots[3][SEGMENT_ROWS];
    const int64_t t = blockIdx.x, nt = gridDim.x;
    const int seg = blockIdx.y, rows = min(SEGMENT_ROWS, a.K - seg * SEGMENT_ROWS), tid = threadIdx.x, lane = tid & 63;
    load_tile(a, t, seg, tile);
    if (seg == 0) {
        const uint32_t* const from = (const uint32_t*)a.heads;
        for (int64_t i = t * THREADS + tid; i < a.head_dwords + a.wide_head_dwords; i += nt * THREADS)
            (i < a.head_dwords ? (uint32_t*)a.weight + i : (uint32_t*)a.wide + (i - a.head_dwords))[0] = from[i];
    }
    __syncthreads();
    find_masks(a.n4, tile, mask);
    int first[3] = {0, 0, 0}, count[3] = {0, 0, 0};
    for (int i = 0; i < 3; ++i) {
        const int64_t of = i == 2 ? t : 2 * t + i;
        if (i == 2 ? a.wide == nullptr : of >= a.ntiles) continue;
        const int32_t* const bounds =
            (const int32_t*)(a.heads + (i == 2 ? 4 * a.head_dwords + wide_bounds_offset(nt) : bounds_offset(a.ntiles))) + of * (a.nseg + 1);
        first[i] = bounds[seg];
        count[i] = bounds[seg + 1] - first[i];
        const int16_t* const from = (i == 2 ? a.wide_slots : a.slots) + (of * a.nseg + seg) * SEGMENT_ROWS;
        for (int z = tid; z < count[i] * STEP_K; z += THREADS) slots[i][z] = from[z];
        const int room = i == 2 ? a.wide_tile_steps : a.tile_steps;
        if (seg == a.nseg - 1 && room) {
            const int64_t past = bounds[a.nseg], size = i == 2 ? WIDE_RECORD_BYTES : RECORD_BYTES;
            clear_records((i == 2 ? a.wide + wide_records_offset(nt, a.nseg) : a.weight + records_offset(a.ntiles, a.nseg)) + past * size,
                          ((of + 1) * room - past) * size);
        }
    }
    __syncthreads();
    // row tiles: lane 16 g + row has the values of slots 16 g .. 16 g + 15
    for (int i = 0; i < 2; ++i) {
        const uint8_t* const row = tile + (16 * i + (lane & 15)) * PITCH;
        for (int s = tid >> 6; s < count[i]; s += THREADS / 64) {
            uint8_t* const rec = a.weight + records_offset(a.ntiles, a.nseg) + (int64_t)(first[i] + s) * RECORD_BYTES;
            const int16_t* const slot = slots[i] + s * STEP_K;
            v4i v = {0, 0, 0, 0};
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int k = slot[(lane & 48) + j];
                if (k >= 0) v[j >> 2] |= (int)((uint32_t)row[k] << (8 * (j & 3)));
            }
            *(v4i*)(rec + 16 * lane) = v;
            if (lane < STEP_IDX_DWORDS) {
                const int z = 16 * (lane >> 3) + (lane & 7), k0 = slot[z], k1 = slot[z + 8];
                const uint32_t low = (uint32_t)(seg * SEGMENT_ROWS + (k0 < 0 ? ~k0 : k0)), high = (uint32_t)(seg * SEGMENT_ROWS + (k1 < 0 ? ~k1 : k1));
                *(uint32_t*)(rec + STEP_VAL_BYTES + 4 * lane) = low | high << 16;
            }
        }
    }
    // wide tile: lane 32 h + row has two values of each quad of slots 16 h .. 16 h + 15 and 32 + 16 h .., and where they are in it
    for (int s = tid >> 6; s < count[2]; s += THREADS / 64) {
        uint8_t* const rec = a.wide + wide_records_offset(nt, a.nseg) + (int64_t)(first[2] + s) * WIDE_RECORD_BYTES;
        const int16_t* const slot = slots[2] + s * STEP_K;
        const int h = lane >> 5, r = lane & 31, unit = a.n4 ? r >> 2 : r;
        v4i v = {0, 0, 0, 0};
        uint32_t sel = 0;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int z0 = 32 * (q >> 2) + 16 * h + 4 * (q & 3);
            int have = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int k = slot[z0 + j];
                if (k >= 0 && (mask[k] >> unit & 1)) {
                    const int at = 2 * q + have;           // (of the 16 values; have: 0 or 1)
                    const uint32_t byte = tile[r * PITCH + k];
                    v[q >> 1] |= (int)(byte << (8 * (at & 3)));
                    sel |= (uint32_t)j << (2 * at);
                    have = 1;
                }
            }
        }
        *(v4i*)(rec + 16 * lane) = v;
        const int z = 32 * h + 16 * (lane & 1) + ((lane & 15) >> 1);
        auto row_of = [&](const int z) {
            const int k = slot[z], pad = ((z & 7) + (z >> 3)) & 7;
            return 32u * (uint32_t)(k >= 0 ? k : pad < rows ? pad : 0);
        };
        uint32_t* const more = (uint32_t*)(rec + WIDE_VAL_BYTES + 8 * lane);
        more[0] = sel;
        more[1] = row_of(z) | row_of(z + 8) << 16;
    }
}

// By its address, which returns the launch's own error: the one that the runtime keeps may be of any earlier call that failed, and
// stays for whoever asks for it.
hipError_t launch(void (*kernel)(PackArgs), int64_t nt, int64_t nseg, const PackArgs& a)
{
    const void* args[] = {&a};
    return hipLaunchKernel((const void*)kernel, dim3((unsigned)nt, (unsigned)nseg), dim3(THREADS), (void**)args, 0, nullptr);
}

constexpr int64_t up(int64_t bytes) { return (bytes + 255) & ~(int64_t)255; }

}  // namespace

DevicePack::~DevicePack() { (void)give_back(); }

// (hipFree waits for all streams of the device, also for those that the default stream does not wait for: 45 ms of a program's other
// work were in the pack.  Freed in the default stream's order the memory goes back when that stream has been waited for: until then
// the pool keeps it, as large as the weight.  This takes up to 10 us more than hipFree: packed, unpacked and released, 1024x1024 at 80 %
// 285 -> 295 us, 1024x4096 562 -> 567.)
int DevicePack::give_back()
{
    if (!scratch_) return hipSuccess;
    (void)hipFreeAsync(scratch_, nullptr);
    scratch_ = nullptr;
    return hipStreamSynchronize(nullptr);
}

bool DevicePack::reserve(int64_t N, int64_t K, spmm_block_t block)
{
    N_ = N;
    K_ = K;
    n4_ = block == SPMM_BLOCK_N4K1;
    nseg_ = (K + SEGMENT_ROWS - 1) / SEGMENT_ROWS;
    ntiles_ = (N + TILE_ROWS - 1) / TILE_ROWS;
    nt_ = (ntiles_ + 1) / 2;
    info_at_ = up(N * K);
    slots_at_ = info_at_ + up((ntiles_ + nt_ * (1 + WIDE_ROWS)) * nseg_ * 4);
    wide_slots_at_ = slots_at_ + up(ntiles_ * nseg_ * SEGMENT_ROWS * 2);
    heads_at_ = wide_slots_at_ + up(nt_ * nseg_ * SEGMENT_ROWS * 2);
    const int64_t size = heads_at_ + records_offset(ntiles_, nseg_) + RECORD_BYTES + wide_records_offset(nt_, nseg_) + WIDE_RECORD_BYTES;
    if (hipMallocAsync((void**)&scratch_, (size_t)size, nullptr) == hipSuccess) return true;
    scratch_ = nullptr;
    (void)hipGetLastError();
    return false;
}

void DevicePack::begin(const int8_t* W)
{
    error_ = hipMemcpy(scratch_, W, (size_t)(N_ * K_), hipMemcpyHostToDevice);
    if (error_ != hipSuccess) return;
    PackArgs a = {};
    a.W = (const int8_t*)scratch_;
    a.info = (int32_t*)(scratch_ + info_at_);
    a.slots = (int16_t*)(scratch_ + slots_at_);
    a.wide_slots = (int16_t*)(scratch_ + wide_slots_at_);
    a.N = N_;
    a.K = (int)K_;
    a.nseg = (int)nseg_;
    a.ntiles = (int)ntiles_;
    a.n4 = n4_;
    error_ = launch(spmm_pack_lists, nt_, nseg_, a);
}

int DevicePack::finish(HostLayout& hl, DeviceForms& f, uint8_t** weight)
{
    const int64_t numbers = (ntiles_ + nt_ * (1 + WIDE_ROWS)) * nseg_;
    const std::unique_ptr<int32_t[]> info(new int32_t[(size_t)numbers]);
    hipError_t e = (hipError_t)error_;
    if (e == hipSuccess) e = hipMemcpy(info.get(), scratch_ + info_at_, (size_t)(numbers * 4), hipMemcpyDeviceToHost);
    if (e == hipSuccess) {
        std::vector<uint8_t> heads;
        int64_t head = 0;
        dims_from_steps(N_, K_, info.get(), info.get() + ntiles_ * nseg_, info.get() + (ntiles_ + nt_) * nseg_, hl, f, heads, head);
        e = hipMalloc((void**)weight, (size_t)(f.size + f.wide_size));
        if (e != hipSuccess) *weight = nullptr;
        if (e == hipSuccess) e = hipMemcpy(scratch_ + heads_at_, heads.data(), heads.size(), hipMemcpyHostToDevice);
        if (e == hipSuccess) {
            PackArgs a = {};
            a.W = (const int8_t*)scratch_;
            a.slots = (int16_t*)(scratch_ + slots_at_);
            a.wide_slots = (int16_t*)(scratch_ + wide_slots_at_);
            a.heads = scratch_ + heads_at_;
            a.head_dwords = head / 4;
            a.wide_head_dwords = ((int64_t)heads.size() - head) / 4;
            a.weight = *weight;
            a.wide = f.wide_size ? *weight + f.size : nullptr;
            a.N = N_;
            a.K = (int)K_;
            a.nseg = (int)nseg_;
            a.ntiles = (int)ntiles_;
            a.tile_steps = f.tile_steps;
            a.wide_tile_steps = f.wide_tile_steps;
            a.n4 = n4_;
            e = launch(spmm_pack_records, nt_, nseg_, a);
        }
    }
    const hipError_t done = (hipError_t)give_back();        // (and the weight is there for every stream when the call returns)
    if (e == hipSuccess) e = done;
    if (e != hipSuccess) {
        if (*weight) (void)hipFree(*weight);        // (the host may pack instead, into an allocation of its own)
        *weight = nullptr;
        (void)hipGetLastError();
    }
    return e;
}

}  // namespace spmm
