// Host-side packer: dense-with-zeros int8 weight -> canonical 4x1 block-sparse rows ->
// the device's row-tile union layout (see spmm_internal.h).  Pure C++, no GPU calls.
//
// Paper Section 3.1 / Figure 1: blocks of 4x1 with the sparsity dimension on the output
// channels.  Section 3.2: the kernel is specialised on the sparse weight and its indices,
// and the block count is padded to what the multiply instruction accumulates over (note
// after Algorithm 1).  Here that instruction is the 16x16x64 int8 matrix op, so the unit
// of padding is 64 listed k positions per 16-row tile.
#include <algorithm>
#include <cstring>
#include <memory>

#include "spmm_internal.h"
#include "team.h"

namespace spmm {

namespace {

inline uint64_t load8(const int8_t* p)
{
    uint64_t v;
    std::memcpy(&v, p, 8);
    return v;
}

// bit i: byte i is not zero
inline uint64_t nonzero_bytes(uint64_t v)
{
    const uint64_t high = (((v & 0x7f7f7f7f7f7f7f7full) + 0x7f7f7f7f7f7f7f7full) | v) & 0x8080808080808080ull;
    return (high >> 7) * 0x0102040810204080ull >> 56;
}

// how many blocks block-row br has
int64_t count_blocks_of_row(const int8_t* W, int64_t N, int64_t K, int64_t ldw, spmm_block_t block, int64_t br)
{
    int64_t n = 0;
    if (block == SPMM_BLOCK_N4K1) {
        const int rows = (int)std::min<int64_t>(4, N - br * 4);
        const int8_t* r[4];
        for (int i = 0; i < 4; ++i) r[i] = W + (br * 4 + std::min(i, rows - 1)) * ldw;     // (missing rows: the last one again)
        const int8_t *const r0 = r[0], *const r1 = r[1], *const r2 = r[2], *const r3 = r[3];
        for (int64_t k0 = 0; k0 < K; k0 += 128) {       // (in bytes, which the compiler takes 16 at a time)
            uint8_t some = 0;
            for (int64_t k = k0; k < std::min(K, k0 + 128); ++k) some = (uint8_t)(some + ((r0[k] | r1[k] | r2[k] | r3[k]) != 0));
            n += some;
        }
    } else {
        // (whole blocks on their own: with the length of the last one in question at every block, the canonical form of 256x256
        // at 80 % took 159 us instead of 22, and 102 in a single pass)
        const int8_t* const r = W + br * ldw;
        const int64_t whole = K / 4;
        for (int64_t c0 = 0; c0 < whole; c0 += 1024) {
            uint32_t some = 0;
            for (int64_t c = c0; c < std::min(whole, c0 + 1024); ++c) {
                uint32_t v;
                std::memcpy(&v, r + 4 * c, 4);
                some += v != 0;
            }
            n += some;
        }
        uint32_t v = 0;
        std::memcpy(&v, r + 4 * whole, (size_t)(K - 4 * whole));
        n += v != 0;
    }
    return n;
}

// The blocks of block-row br to index / vals (4 bytes per block)
void blocks_of_row(const int8_t* W, int64_t N, int64_t K, int64_t ldw, spmm_block_t block, int64_t br, int32_t* index, int8_t* vals)
{
    int64_t n = 0;
    if (block == SPMM_BLOCK_N4K1) {
        const int rows = (int)std::min<int64_t>(4, N - br * 4);
        const int8_t* r[4];
        for (int i = 0; i < 4; ++i) r[i] = W + (br * 4 + std::min(i, rows - 1)) * ldw;     // (missing rows: the last one again)
        const uint32_t keep = rows == 4 ? 0xffffffffu : (1u << (8 * rows)) - 1u;
        auto add = [&](int64_t k) {
            const uint32_t v = ((uint32_t)(uint8_t)r[0][k] | (uint32_t)(uint8_t)r[1][k] << 8 | (uint32_t)(uint8_t)r[2][k] << 16 |
                                (uint32_t)(uint8_t)r[3][k] << 24) & keep;
            index[n] = (int32_t)k;
            std::memcpy(vals + 4 * n++, &v, 4);
        };
        int64_t k = 0;
        for (; k + 64 <= K; k += 64) {      // 64 positions at a time: few mispredicted loop ends
            uint64_t m = 0;
            for (int i = 0; i < 8; ++i) {
                const int64_t at = k + 8 * i;
                m |= nonzero_bytes(load8(r[0] + at) | load8(r[1] + at) | load8(r[2] + at) | load8(r[3] + at)) << (8 * i);
            }
            for (; m; m &= m - 1) add(k + __builtin_ctzll(m));
        }
        for (; k < K; ++k)
            if (r[0][k] | r[1][k] | r[2][k] | r[3][k]) add(k);
    } else {
        const int8_t* r = W + br * ldw;
        const int64_t whole = K / 4;
        auto add = [&](int64_t c, uint32_t v) {
            if (!v) return;
            index[n] = (int32_t)c;
            std::memcpy(vals + 4 * n++, &v, 4);
        };
        uint32_t v;
        for (int64_t c = 0; c < whole; ++c) {
            std::memcpy(&v, r + 4 * c, 4);
            add(c, v);
        }
        v = 0;
        std::memcpy(&v, r + 4 * whole, (size_t)(K - 4 * whole));
        add(whole, v);
    }
}

}  // namespace

void bsr_from_dense(const int8_t* W, int64_t N, int64_t K, int64_t ldw, spmm_block_t block, Bsr& out)
{
    Team team;
    bsr_from_dense(W, N, K, ldw, block, out, team);
}

// Two passes over the weight: how many blocks there are, and the blocks, to where they stay.  (In one, with pieces put together
// afterwards, every block was written twice, to new pages both times: 1024x4096 at 80 %, 220 to 270 us, now 180.)
void bsr_from_dense(const int8_t* W, int64_t N, int64_t K, int64_t ldw, spmm_block_t block, Bsr& out, Team& team, const Beside* beside)
{
    out.N = N;
    out.K = K;
    out.block = block;
    out.block_rows = (block == SPMM_BLOCK_N4K1) ? (N + 3) / 4 : N;
    out.row_ptr.assign((size_t)out.block_rows + 1, 0);
    const int64_t rows_per_block_row = (block == SPMM_BLOCK_N4K1) ? 4 : 1;
    const int64_t piece = std::max<int64_t>(1, 65536 / (K * rows_per_block_row));
    team.run(out.block_rows, piece, [&](int64_t begin, int64_t end) {
        for (int64_t br = begin; br < end; ++br) out.row_ptr[(size_t)br + 1] = count_blocks_of_row(W, N, K, ldw, block, br);
    }, [&] { if (beside) beside->first(); });
    for (int64_t br = 0; br < out.block_rows; ++br) out.row_ptr[(size_t)br + 1] += out.row_ptr[(size_t)br];
    out.index.resize((size_t)out.row_ptr.back());
    out.vals.resize((size_t)out.row_ptr.back() * 4);
    auto fill = [&](int64_t begin, int64_t end) {
        for (int64_t br = begin; br < end; ++br) {
            const size_t at = (size_t)out.row_ptr[(size_t)br];
            blocks_of_row(W, N, K, ldw, block, br, out.index.data() + at, out.vals.data() + 4 * at);
        }
    };
    if (beside) team.finish(out.block_rows, piece, fill, beside->last);
    else team.run(out.block_rows, piece, fill);
}

void bsr_to_dense(const Bsr& b, int8_t* W, int64_t ldw)
{
    const bool n4 = b.block == SPMM_BLOCK_N4K1;
    Team team;
    team.finish(b.block_rows, std::max<int64_t>(1, 262144 / (b.K * (n4 ? 4 : 1))), [&](int64_t begin, int64_t end) {
        for (int64_t br = begin; br < end; ++br) {
            const int rows = n4 ? (int)std::min<int64_t>(4, b.N - br * 4) : 1;
            int8_t* const w = W + br * (n4 ? 4 : 1) * ldw;
            for (int i = 0; i < rows; ++i) std::memset(w + i * ldw, 0, (size_t)b.K);
            for (int64_t e = b.row_ptr[(size_t)br]; e < b.row_ptr[(size_t)br + 1]; ++e) {
                const int8_t* v = &b.vals[(size_t)e * 4];
                if (n4) {
                    const int64_t k = b.index[(size_t)e];
                    for (int i = 0; i < rows; ++i) w[i * ldw + k] = v[i];
                } else {
                    const int64_t k0 = (int64_t)b.index[(size_t)e] * 4;
                    std::memcpy(w + k0, v, (size_t)std::min<int64_t>(4, b.K - k0));
                }
            }
        }
    });
}

// Order the listed k of one (row tile, segment) inside its steps so that the transposing
// LDS reads hit distinct banks.
//
// One ds_read_b64_tr_b8 of a wave touches 32 activation rows (4 lane groups x 8 rows), 16 bytes
// each; with the row pitch used by the kernels (token tile + 16 bytes) a row starts at LDS
// bank 4 * ((9 * row) % 16), so two rows collide exactly when their indices are congruent
// mod 16.  The 64 slots of a step are read by two instructions (slots t < 8 and t >= 8 of
// every group), each in two half-waves (groups {0,1} and {2,3}): four "half-reads" of 16 rows.
// The entries are dealt out so that a half-read holds every residue mod 16 at most once
// whenever the counts allow it; padding slots (zero weights) are pointed at a row of a
// residue the half-read still lacks instead of all hitting row 0.
// place(k, slot, row) is called for every slot of the steps once: k = -1 is padding, row the row that it reads.
template <typename P>
static void arrange_for_lds_banks(const uint32_t* mask, const uint32_t mine, int rows, int nsteps, const P& place)
{
    if (nsteps == 0) return;
    const int H = 4 * nsteps;                           // half-reads, at most 32
    // entries by residue
    int16_t by_res[16][SEGMENT_ROWS / 16 + 1];
    int n_res[16] = {0}, order[16];
    for (int k = 0; k < rows; ++k) {
        by_res[k & 15][n_res[k & 15]] = (int16_t)k;
        n_res[k & 15] += (mask[k] & mine) != 0;
    }
    for (int r = 0; r < 16; ++r) {                      // largest class first, stable
        int i = r;
        for (; i > 0 && n_res[order[i - 1]] < n_res[r]; --i) order[i] = order[i - 1];
        order[i] = r;
    }
    // Largest residue class first; each class is spread over the least-filled half-reads, one entry per half-read, so that
    // no half-read runs out of room while others still have holes.  Only a class with more than H entries is forced to
    // double up somewhere.  Filled that way, the half-reads hold `load` entries (those in `low`) or one more.
    const uint32_t all = H == 32 ? ~0u : (1u << H) - 1;
    uint32_t low = all, present[32] = {0};
    int load = 0;
    auto slot_of = [](int h, int j) { return h / 4 * STEP_K + 16 * (2 * (h & 1) + j / 8) + 8 * (h / 2 % 2) + j % 8; };
    for (int oi = 0; oi < 16; ++oi) {
        const int r = order[oi];
        int next = 0;
        auto deal = [&](uint32_t to, int j) {           // an entry to each, in order; those that had none left are returned
            for (; to && next < n_res[r]; to &= to - 1) {
                const int h = __builtin_ctz(to), k = by_res[r][next++];
                present[h] |= 1u << r;
                place(k, slot_of(h, j), k);
            }
            return to;
        };
        while (next < n_res[r]) {
            const uint32_t high = all & ~low, left = deal(low, load);
            if (left) {
                low = left;
            } else {
                const uint32_t still = deal(high, load + 1);
                low |= still;
                ++load;
                if (!low) {                             // (cannot be: `low` was not empty)
                    low = all;
                    ++load;
                }
            }
        }
    }
    for (int h = 0; h < H; ++h) {
        int next_res = 0;
        for (int j = load + !(low >> h & 1); j < 16; ++j) {
            while (next_res < 16 && (present[h] & (1u << next_res))) ++next_res;
            int row = 0;
            if (next_res < 16) {
                if (next_res < rows) row = next_res;
                present[h] |= 1u << next_res;
            }
            place(-1, slot_of(h, j), row);
        }
    }
}

// ---------------------------------------------------------------------------------------
// Offline ordering of the output rows (Section 3.2: what can be tuned offline for a given
// sparse weight).  A row tile multiplies the UNION of the k lists of its rows, padded to
// whole steps, so rows with similar lists belong in one tile.  The movable unit is what
// keeps the block structure: a 4x1 block-row (four consecutive rows) in the paper's
// orientation, a single row for 1x4 blocks; a trailing partial block-row stays last, so the
// first N rows of the new order are exactly the N rows of the weight.
//
// Greedy clustering: units are taken heaviest first; a tile is opened with the heaviest
// unit left and filled with the units (among the next `window` in that order) that add the
// fewest steps, then the fewest listed k, to the tile's per-segment unions.  Heaviest-first
// also puts rows of similar length next to each other, which is what the waves of one
// workgroup (one row tile each, in lock-step per segment) want.
// ---------------------------------------------------------------------------------------
namespace {

struct KSet {
    std::vector<uint64_t> w;   // one bit per k
};

inline int popcount64(uint64_t x) { return __builtin_popcountll(x); }

// steps of a union, per segment of kc (a multiple of 64) positions
int64_t steps_of(const std::vector<uint64_t>& u, int words_per_seg, int64_t* listed)
{
    int64_t steps = 0, total = 0;
    for (size_t w0 = 0; w0 < u.size(); w0 += (size_t)words_per_seg) {
        int cnt = 0;
        for (size_t w = w0; w < std::min(u.size(), w0 + (size_t)words_per_seg); ++w) cnt += popcount64(u[w]);
        steps += (cnt + STEP_K - 1) / STEP_K;
        total += cnt;
    }
    if (listed) *listed = total;
    return steps;
}

}  // namespace

void order_rows_by_k_overlap(const Bsr& b, int kc, std::vector<int32_t>& row_order)
{
    const bool n4 = (b.block == SPMM_BLOCK_N4K1);
    const int unit_rows = n4 ? 4 : 1;
    const int group = TILE_ROWS / unit_rows;             // units per row tile
    const int64_t full_units = n4 ? b.N / 4 : b.N;       // a trailing partial block-row is not moved
    const int words = (int)((b.K + 63) / 64), words_per_seg = kc / 64;

    std::vector<KSet> ks((size_t)full_units);
    std::vector<int64_t> weight((size_t)full_units);
    for (int64_t u = 0; u < full_units; ++u) {
        ks[(size_t)u].w.assign((size_t)words, 0);
        weight[(size_t)u] = b.row_ptr[u + 1] - b.row_ptr[u];
        for (int64_t e = b.row_ptr[u]; e < b.row_ptr[u + 1]; ++e) {
            if (n4) {
                const int64_t k = b.index[e];
                ks[(size_t)u].w[(size_t)(k >> 6)] |= (uint64_t)1 << (k & 63);
            } else {
                for (int j = 0; j < 4; ++j) {
                    const int64_t k = (int64_t)b.index[e] * 4 + j;
                    if (k < b.K) ks[(size_t)u].w[(size_t)(k >> 6)] |= (uint64_t)1 << (k & 63);
                }
            }
        }
    }
    std::vector<int64_t> by_weight((size_t)full_units);
    for (int64_t u = 0; u < full_units; ++u) by_weight[(size_t)u] = u;
    std::stable_sort(by_weight.begin(), by_weight.end(),
                     [&](int64_t x, int64_t y) { return weight[(size_t)x] > weight[(size_t)y]; });

    const int64_t window = 512;
    std::vector<char> used((size_t)full_units, 0);
    std::vector<int64_t> unit_order;
    unit_order.reserve((size_t)full_units);
    std::vector<uint64_t> uni((size_t)words), trial((size_t)words);
    int64_t first_free = 0;   // position in by_weight of the heaviest unit not yet placed
    while ((int64_t)unit_order.size() < full_units) {
        while (used[(size_t)by_weight[(size_t)first_free]]) ++first_free;
        const int64_t seed = by_weight[(size_t)first_free];
        used[(size_t)seed] = 1;
        unit_order.push_back(seed);
        uni = ks[(size_t)seed].w;
        for (int slot = 1; slot < group && (int64_t)unit_order.size() < full_units; ++slot) {
            int64_t best = -1, best_steps = 0, best_listed = 0, seen = 0;
            for (int64_t p = first_free; p < full_units && seen < window; ++p) {
                const int64_t u = by_weight[(size_t)p];
                if (used[(size_t)u]) continue;
                ++seen;
                for (int w = 0; w < words; ++w) trial[(size_t)w] = uni[(size_t)w] | ks[(size_t)u].w[(size_t)w];
                int64_t listed = 0;
                const int64_t st = steps_of(trial, words_per_seg, &listed);
                if (best < 0 || st < best_steps || (st == best_steps && listed < best_listed)) {
                    best = u; best_steps = st; best_listed = listed;
                }
            }
            used[(size_t)best] = 1;
            unit_order.push_back(best);
            for (int w = 0; w < words; ++w) uni[(size_t)w] |= ks[(size_t)best].w[(size_t)w];
        }
    }
    row_order.clear();
    row_order.reserve((size_t)b.N);
    for (const int64_t u : unit_order)
        for (int i = 0; i < unit_rows; ++i) row_order.push_back((int32_t)(u * unit_rows + i));
    for (int64_t n = full_units * unit_rows; n < b.N; ++n) row_order.push_back((int32_t)n);   // the partial block-row
}

// The weight with its rows in the given order (whole units, see above), as a canonical form of its own.
void bsr_permute_rows(const Bsr& b, const std::vector<int32_t>& row_order, Bsr& out)
{
    const int unit_rows = (b.block == SPMM_BLOCK_N4K1) ? 4 : 1;
    out.N = b.N; out.K = b.K; out.block = b.block; out.block_rows = b.block_rows;
    out.row_ptr.assign(1, 0);
    out.index.clear(); out.vals.clear();
    out.index.reserve(b.index.size()); out.vals.reserve(b.vals.size());
    for (int64_t br = 0; br < b.block_rows; ++br) {
        const int64_t src = row_order[(size_t)(br * unit_rows)] / unit_rows;
        out.index.insert(out.index.end(), b.index.begin() + b.row_ptr[src], b.index.begin() + b.row_ptr[src + 1]);
        out.vals.insert(out.vals.end(), b.vals.begin() + 4 * b.row_ptr[src], b.vals.begin() + 4 * b.row_ptr[src + 1]);
        out.row_ptr.push_back((int64_t)out.index.size());
    }
}

// ---------------------------------------------------------------------------------------
// Both layouts start from the lists of 32 rows: which of their units (block-rows, or rows of 1x4 blocks) list a k.
// ---------------------------------------------------------------------------------------
namespace {

struct Lists {
    const Bsr& b;
    const bool n4;
    const int64_t K;
    const int units;                        // of a wide tile; half as many of a row tile
    const uint32_t half;                    // the units of a wide tile's first row tile
    const int nseg, ntiles;
    const int64_t nt, grain;                // wide tiles; and of them, how many make a piece of work
    std::unique_ptr<uint32_t[]> masks;      // [wide tile][k]: the units that list k
    std::vector<int32_t> steps, wide_steps; // of every (row tile, segment); of every (wide tile, segment), if none needs more

    // (rows past N and block-rows past the end list nothing)
    Lists(const Bsr& bsr, int32_t* rowsum, Team& team)
        : b(bsr), n4(b.block == SPMM_BLOCK_N4K1), K(b.K), units(n4 ? WIDE_ROWS / 4 : WIDE_ROWS), half(n4 ? 0xfu : 0xffffu),
          nseg((int)((K + SEGMENT_ROWS - 1) / SEGMENT_ROWS)), ntiles((int)((b.N + TILE_ROWS - 1) / TILE_ROWS)), nt((ntiles + 1) / 2),
          grain(std::max<int64_t>(1, 65536 / (K * WIDE_ROWS))), masks(new uint32_t[(size_t)(nt * K)]), steps((size_t)ntiles * nseg),
          wide_steps((size_t)nt * nseg)
    {
        team.run(nt, grain, [&](int64_t begin, int64_t end) {
            for (int64_t t = begin; t < end; ++t) {
                uint32_t* const mask = &masks[(size_t)(t * K)];
                std::memset(mask, 0, (size_t)K * 4);
                for (int u = 0; u < units && t * units + u < b.block_rows; ++u) {
                    const int64_t first = b.row_ptr[(size_t)(t * units + u)], past = b.row_ptr[(size_t)(t * units + u + 1)];
                    const int32_t* const index = b.index.data();
                    const int8_t* const v = b.vals.data();
                    const uint32_t bit = 1u << u;
                    int32_t sum[4] = {0, 0, 0, 0};
                    for (int64_t e = first; e < past; ++e)
                        for (int j = 0; j < 4; ++j) sum[j] += v[4 * e + j];
                    if (n4) {
                        for (int64_t e = first; e < past; ++e) mask[index[e]] |= bit;
                        for (int j = 0; j < 4; ++j)
                            if (t * WIDE_ROWS + 4 * u + j < (int64_t)ntiles * TILE_ROWS) rowsum[t * WIDE_ROWS + 4 * u + j] = sum[j];
                    } else {
                        for (int64_t e = first; e < past; ++e)
                            for (int j = 0; j < 4; ++j)
                                if (v[4 * e + j]) mask[index[e] * 4 + j] |= bit;
                        rowsum[t * WIDE_ROWS + u] = sum[0] + sum[1] + sum[2] + sum[3];
                    }
                }
                for (int seg = 0; seg < nseg; ++seg) {
                    const int rows = rows_of(seg);
                    const uint32_t* const m = mask + seg * SEGMENT_ROWS;
                    int all = 0, low = 0, high = 0;
                    for (int k = 0; k < rows; ++k) {
                        all += m[k] != 0;
                        low += (m[k] & half) != 0;
                        high += (m[k] & ~half) != 0;
                    }
                    wide_steps[(size_t)(t * nseg + seg)] = (all + STEP_K - 1) / STEP_K;
                    steps[(size_t)(2 * t * nseg + seg)] = (low + STEP_K - 1) / STEP_K;
                    if (2 * t + 1 < ntiles) steps[(size_t)((2 * t + 1) * nseg + seg)] = (high + STEP_K - 1) / STEP_K;
                }
            }
        });
    }
    int rows_of(int seg) const { return (int)std::min<int64_t>(SEGMENT_ROWS, K - (int64_t)seg * SEGMENT_ROWS); }
};

// The steps of a row tile: listed k dealt to slots, every block's values scattered to their lanes (vals[step][lane = 16 g +
// row][t] of slot 16 g + t).  The values of a step and its positions lie `stride` bytes from those of the step before; `place`
// is scratch of K numbers; positions are relative to the segment, or to the weight.
void arrange_tile(const Lists& l, int64_t tile, uint8_t* vals, int64_t val_stride, uint8_t* idx, int64_t idx_stride, bool of_weight,
                  int32_t* place)
{
    const Bsr& b = l.b;
    const uint32_t* const mask = &l.masks[(size_t)(tile / 2 * l.K)];
    const uint32_t mine = tile & 1 ? ~l.half : l.half;
    int step = 0;
    for (int seg = 0; seg < l.nseg; ++seg) {
        const int k_lo = seg * SEGMENT_ROWS, rows = l.rows_of(seg), count = l.steps[(size_t)(tile * l.nseg + seg)];
        const int base = of_weight ? k_lo : 0;
        arrange_for_lds_banks(mask + k_lo, mine, rows, count, [&](int k, int slot, int row) {
            const int t = slot & (STEP_K - 1), s = step + slot / STEP_K;
            if (k >= 0) place[k_lo + k] = (int32_t)(s * val_stride + (t & ~15) * 16 + (t & 15));     // of row 0; row r is 16 r bytes on
            // 8 g + t % 8 of the pairs, low half for slot 16 g + t % 8 and high half for 8 more
            const uint16_t at = (uint16_t)(base + row);
            std::memcpy(idx + s * idx_stride + 4 * (8 * (t >> 4) + (t & 7)) + 2 * (t >> 3 & 1), &at, 2);
        });
        for (int s = 0; s < count; ++s, ++step) std::memset(vals + step * val_stride, 0, STEP_VAL_BYTES);
    }
    const int units = l.units / 2;
    for (int q = 0; q < units && tile * units + q < b.block_rows; ++q) {
        const int64_t br = tile * units + q;
        for (int64_t e = b.row_ptr[(size_t)br]; e < b.row_ptr[(size_t)br + 1]; ++e) {
            uint32_t v;
            std::memcpy(&v, &b.vals[(size_t)e * 4], 4);
            const int32_t at = b.index[(size_t)e];
            if (l.n4) {
                uint8_t* const to = vals + place[at] + 4 * q * 16;
                for (int j = 0; j < 4; ++j) to[16 * j] = (uint8_t)(v >> (8 * j));
            } else {
                for (int j = 0; j < 4; ++j)
                    if (v >> (8 * j) & 0xff) vals[place[at * 4 + j] + q * 16] = (uint8_t)(v >> (8 * j));
            }
        }
    }
}

// dimensions and bounds of the row tiles, from the steps of every (row tile, segment)
void layout_dims(int nseg, int ntiles, const int32_t* steps, HostLayout& out)
{
    out.kc = SEGMENT_ROWS;
    out.nseg = nseg;
    out.ntiles = ntiles;
    out.max_steps_per_tile = 0;
    out.max_steps_per_segment = 0;
    out.seg_ptr.assign((size_t)ntiles * nseg + 1, 0);
    for (int64_t tile = 0; tile < ntiles; ++tile) {
        int steps_this_tile = 0;
        for (int seg = 0; seg < nseg; ++seg) {
            const size_t i = (size_t)(tile * nseg + seg);
            steps_this_tile += steps[i];
            out.max_steps_per_segment = std::max(out.max_steps_per_segment, steps[i]);
            out.seg_ptr[i + 1] = out.seg_ptr[i] + steps[i];
        }
        out.max_steps_per_tile = std::max(out.max_steps_per_tile, steps_this_tile);
    }
    out.nsteps = out.seg_ptr.back();
}

}  // namespace

void layout_from_bsr(const Bsr& b, int kc, HostLayout& out)
{
    Team team;
    layout_from_bsr(b, kc, out, team);
}

void layout_from_bsr(const Bsr& b, int kc, HostLayout& out, Team& team)
{
    (void)kc;                                               // SEGMENT_ROWS
    out.rowsum.assign((size_t)((b.N + TILE_ROWS - 1) / TILE_ROWS) * TILE_ROWS, 0);
    const Lists l(b, out.rowsum.data(), team);
    layout_dims(l.nseg, l.ntiles, l.steps.data(), out);
    out.vals.assign((size_t)out.nsteps * STEP_VAL_BYTES, 0);
    out.idx.assign((size_t)out.nsteps * STEP_IDX_DWORDS, 0);
    team.finish(l.ntiles, 2 * l.grain, [&](int64_t begin, int64_t end) {
        const std::unique_ptr<int32_t[]> place(new int32_t[(size_t)l.K]);
        for (int64_t t = begin; t < end; ++t) {
            const size_t first = (size_t)out.seg_ptr[(size_t)(t * l.nseg)];
            arrange_tile(l, t, out.vals.data() + first * STEP_VAL_BYTES, STEP_VAL_BYTES, (uint8_t*)(out.idx.data() + first * STEP_IDX_DWORDS),
                         4 * STEP_IDX_DWORDS, false, place.get());
        }
    });
}

void export_steps(const HostLayout& hl, const DeviceForms& f, uint8_t* vals, uint32_t* idx)
{
    const int64_t ns = hl.nseg;
    const uint8_t* const rec = f.bytes.get() + records_offset(hl.ntiles, ns);
    for (int64_t t = 0; t < hl.ntiles; ++t) {
        const int64_t shift = f.tile_steps ? t * f.tile_steps - hl.seg_ptr[(size_t)(t * ns)] : 0;
        for (int64_t g = 0; g < ns; ++g)
            for (int64_t s = hl.seg_ptr[(size_t)(t * ns + g)]; s < hl.seg_ptr[(size_t)(t * ns + g + 1)]; ++s) {
                const uint8_t* const r = rec + (s + shift) * RECORD_BYTES;
                if (vals) std::memcpy(vals + s * STEP_VAL_BYTES, r, STEP_VAL_BYTES);
                if (!idx) continue;
                std::memcpy(idx + s * STEP_IDX_DWORDS, r + STEP_VAL_BYTES, 4 * STEP_IDX_DWORDS);
                for (int i = 0; i < STEP_IDX_DWORDS; ++i) idx[s * STEP_IDX_DWORDS + i] -= (uint32_t)(g * SEGMENT_ROWS) * 0x10001u;
            }
    }
}

// ---------------------------------------------------------------------------------------
// The wide form (spmm_internal.h): 32 rows share a list, and of every 4 consecutive slots (a quad) a row may use two.
//
// Two conditions bind the listed k of a segment to slots.  Quads: no unit (block-row, or row of 1x4 blocks) has more than
// two of a quad's k.  Banks: a gather of half a wave reads the 8 activation rows of one octet of slots, 32 bytes each,
// and rows lie 32 bytes apart in LDS, so they hit distinct banks when their residues mod 8 differ.  Both are met by
// dealing, octet by octet, one k of every residue class, the heaviest that still fits its quad.  What is left when a
// class or a fit runs out goes to the holes that remain, by an exchange if need be, and to a new step at the worst.
// (512 random positions at 70 to 90 %, 8 block-rows: no step more than the list's length asks for, and 0 to 9 of 100
// octets with a residue twice; 32 rows of 1x4 blocks at 75 %: 8.4 steps where 8 would hold the list.)
// ---------------------------------------------------------------------------------------
namespace {

inline int set_bits(uint32_t v)
{
    v -= v >> 1 & 0x55555555u;
    v = (v & 0x33333333u) + (v >> 2 & 0x33333333u);
    return (int)(((v + (v >> 4)) & 0x0f0f0f0fu) * 0x01010101u >> 24);
}

// bit 8 i + j to bit 8 j + i
inline uint64_t transposed8x8(uint64_t x)
{
    uint64_t t = (x ^ x >> 7) & 0x00aa00aa00aa00aaull;
    x ^= t ^ t << 7;
    t = (x ^ x >> 14) & 0x0000cccc0000ccccull;
    x ^= t ^ t << 14;
    t = (x ^ x >> 28) & 0x00000000f0f0f0f0ull;
    return x ^ t ^ t << 28;
}

// bit i of words[u]: bit u of masks[i], for the first `count` of 64 masks (those up to the next multiple of 8 are read)
inline void transposed(const uint32_t* masks, int count, int units, uint64_t* words)
{
    for (int u0 = 0; u0 < units; u0 += 8) {
        uint64_t of[8] = {0};
        for (int i = 0; i < count; i += 8) {
            uint64_t block = 0;
            for (int j = 0; j < 8; ++j) block |= (uint64_t)(masks[i + j] >> u0 & 0xff) << (8 * j);
            block = transposed8x8(block);
            for (int u = 0; u < 8; ++u) of[u] |= (block >> (8 * u) & 0xff) << i;
        }
        for (int u = 0; u < 8; ++u) words[u0 + u] = of[u];
    }
}

struct WideSegment {
    int32_t slot[WIDE_MAX_STEPS * STEP_K];      // segment-local k, -1: padding
    int steps;
};

// false: more than WIDE_MAX_STEPS
bool arrange_wide(const uint32_t* mask, int rows, int units, WideSegment& out)
{
    constexpr int CLASSES = 8, MAX_QUADS = WIDE_MAX_STEPS * STEP_K / 4;
    // candidates of every class, heaviest first, and for every unit which of them it uses
    int16_t cand[CLASSES][SEGMENT_ROWS / CLASSES + 1];
    uint32_t users[CLASSES][SEGMENT_ROWS / CLASSES + 1];
    uint64_t alive[CLASSES], uses[CLASSES][32];
    int16_t start[CLASSES][34] = {{0}};
    uint8_t bucket[SEGMENT_ROWS];
    for (int k = 0; k < rows; ++k) ++start[k % CLASSES][bucket[k] = (uint8_t)(33 - set_bits(mask[k]))];
    int n = 0;
    for (int c = 0; c < CLASSES; ++c) {
        int at = 0;
        for (int w = 0; w < 33; ++w) {
            const int count = start[c][w + 1];
            start[c][w + 1] = (int16_t)at;
            at += count;
            if (w == 31) {                              // (w = 32: those that none uses, after all others)
                alive[c] = at == 64 ? ~(uint64_t)0 : ((uint64_t)1 << at) - 1;
                n += at;
            }
        }
    }
    for (int k = 0; k < rows; ++k) {
        const int c = k % CLASSES, at = start[c][bucket[k]]++;
        cand[c][at] = (int16_t)k;
        users[c][at] = mask[k];
    }
    for (int c = 0; c < CLASSES; ++c) {
        const int m = (rows - c + CLASSES - 1) / CLASSES;
        for (int i = m; i < SEGMENT_ROWS / CLASSES; ++i) users[c][i] = 0;
        transposed(users[c], m, units, uses[c]);
    }
    out.steps = (n + STEP_K - 1) / STEP_K;
    uint32_t one[MAX_QUADS] = {0}, two[MAX_QUADS] = {0};       // units with a k, with two, in the quad
    auto put = [&](int slot, int32_t k, uint32_t m) {
        out.slot[slot] = k;
        two[slot / 4] |= one[slot / 4] & m;
        one[slot / 4] |= m;
    };
    for (int i = 0; i < out.steps * STEP_K; ++i) out.slot[i] = -1;
    for (int o = 0; o < out.steps * 8; ++o) {
        for (int j = 0; j < 8; ++j) {
            const int c = (j + o) & 7;
            uint64_t fit = alive[c];
            for (uint32_t u = two[2 * o + j / 4]; u; u &= u - 1) fit &= ~uses[c][__builtin_ctz(u)];
            if (!fit) continue;
            alive[c] &= ~(fit & (0 - fit));
            put(8 * o + j, cand[c][__builtin_ctzll(fit)], users[c][__builtin_ctzll(fit)]);
        }
    }
    // What is left over, into the quads with holes, or by an exchange: a k of another quad into the hole, and this one into its
    // place.  The other k fits quad q if none of its units has two there, and this one's units m fit in its place if each of
    // them that has two in that quad has one of the two in it.  For all slots at once, 64 of a step in a word: the slots whose k
    // unit u uses (a hole: all units), and those in whose quad u has two.  (256x256 in 1x4 blocks at 70 %, 97 tries a tile: 30 us
    // of a tile slot by slot, 11 so.)
    int holes[MAX_QUADS], nholes = 0;
    uint64_t used[WIDE_MAX_STEPS][32], twice[WIDE_MAX_STEPS][32];
    int words = 0;                                  // (steps that these are filled in of, as exchanges come to look at them)
    auto users_at = [&](int z) { return out.slot[z] < 0 ? ~0u : mask[out.slot[z]]; };
    auto fill_in_words = [&] {
        uint32_t of_slot[STEP_K], of_quad[STEP_K];
        for (int i = 0; i < STEP_K; ++i) {
            of_slot[i] = users_at(words * STEP_K + i);
            of_quad[i] = two[words * STEP_K / 4 + i / 4];
        }
        transposed(of_slot, STEP_K, units, used[words]);
        transposed(of_quad, STEP_K, units, twice[words]);
    };
    auto refresh = [&](int z) {                     // slot z, and its quad
        const uint64_t slot_bit = (uint64_t)1 << (z & 63), quad_bits = (uint64_t)15 << (z & 60);
        const uint32_t m = users_at(z), t = two[z / 4];
        for (int u = 0; u < units; ++u) {
            used[z / 64][u] = (used[z / 64][u] & ~slot_bit) | ((0 - (uint64_t)(m >> u & 1)) & slot_bit);
            twice[z / 64][u] = (twice[z / 64][u] & ~quad_bits) | ((0 - (uint64_t)(t >> u & 1)) & quad_bits);
        }
    };
    auto add_quads = [&](int first, int past) {
        for (int q = first; q < past; ++q) {
            bool hole = false;
            for (int z = 4 * q; z < 4 * q + 4; ++z) hole = hole || out.slot[z] < 0;
            if (hole) holes[nholes++] = q;
        }
    };
    add_quads(0, out.steps * 16);
    auto place = [&](int z, int32_t k, uint32_t m) {
        put(z, k, m);
        if (z / STEP_K < words) refresh(z);
    };
    auto fill = [&](int i, int32_t k, uint32_t m) {             // the first hole of quad holes[i]
        int z = 4 * holes[i], left = 0;
        while (out.slot[z] >= 0) ++z;
        place(z, k, m);
        for (z = 4 * holes[i]; z < 4 * holes[i] + 4; ++z) left += out.slot[z] < 0;
        if (!left) std::copy(holes + i + 1, holes + nholes--, holes + i);
    };
    int exchanges = 256;                            // (a bound on the work; then a new step)
    for (int c = 0; c < CLASSES; ++c) {
        while (alive[c]) {
            const int32_t k = cand[c][__builtin_ctzll(alive[c])];
            const uint32_t m = mask[k];
            bool done = false;
            for (int i = 0; i < nholes && !done; ++i)
                if (!(two[holes[i]] & m)) {
                    fill(i, k, m);
                    done = true;
                }
            uint64_t no_room[WIDE_MAX_STEPS];       // the slots in whose place it does not fit, of the first `looked` steps
            int looked = 0;
            for (int i = 0; i < nholes && !done && exchanges-- > 0; ++i) {
                const int q = holes[i];
                for (int s = 0; s < out.steps && !done; ++s) {
                    for (; words <= s; ++words) fill_in_words();
                    if (looked == s) {
                        no_room[looked++] = 0;
                        for (uint32_t u = m; u; u &= u - 1) no_room[s] |= twice[s][__builtin_ctz(u)] & ~used[s][__builtin_ctz(u)];
                    }
                    uint64_t no = no_room[s] | (s == q / 16 ? (uint64_t)15 << (4 * (q & 15)) : 0);
                    for (uint32_t u = two[q]; u; u &= u - 1) no |= used[s][__builtin_ctz(u)];
                    if (!~no) continue;
                    const int z = s * STEP_K + __builtin_ctzll(~no), r = z / 4;
                    const int32_t other = out.slot[z];
                    const uint32_t u = mask[other];
                    one[r] = (one[r] & ~u) | (two[r] & u);
                    two[r] &= ~u;
                    fill(i, other, u);
                    place(z, k, m);
                    done = true;
                }
            }
            if (!done) {
                if (out.steps == WIDE_MAX_STEPS) return false;
                for (int z = 0; z < STEP_K; ++z) out.slot[out.steps * STEP_K + z] = -1;
                ++out.steps;
                add_quads(out.steps * 16 - 16, out.steps * 16);
                continue;                           // (and again, now that there are holes)
            }
            alive[c] &= alive[c] - 1;
        }
    }
    return true;
}

}  // namespace

namespace {

// activation row of slot z of a record, at the lanes that gather it
inline void set_row(uint8_t* record, int z, int row)
{
    uint16_t* const r = (uint16_t*)(record + WIDE_VAL_BYTES);
    const int lane = 32 * (z >> 5) + 2 * (z & 7) + (z >> 4 & 1), half = z >> 3 & 1;
    r[4 * lane + 2 + half] = r[4 * (lane + 16) + 2 + half] = (uint16_t)(32 * row);
}

// where a listed k has its values in the records of its tile: of row 0, in the first of the two stored; its slot's selector and
// where that goes; and the units whose other stored value is in an earlier slot of the quad
struct WidePlace {
    uint32_t at, before;
    uint16_t sel_word;      // 2 * step + h
    uint8_t sel, shift;
};

// The listed k of a wide tile dealt to the slots of its segments, whose steps go to `steps`.  false: a segment has too many.
// `longer`: in some segment they are more than steps[] had, what the list's length asks for.
bool arrange_segments(const Lists& l, int64_t t, WideSegment* segments, int32_t* steps, bool& longer)
{
    for (int seg = 0; seg < l.nseg; ++seg) {
        if (!arrange_wide(&l.masks[(size_t)(t * l.K + (int64_t)seg * SEGMENT_ROWS)], l.rows_of(seg), l.units, segments[seg])) return false;
        longer = longer || segments[seg].steps > steps[seg];
        steps[seg] = segments[seg].steps;
    }
    return true;
}

// The records of a wide tile so arranged, `room` of them (the last unused ones cleared).
void write_wide_tile(const Lists& l, int64_t t, const WideSegment* segments, uint8_t* rec, int64_t room, WidePlace* places, uint32_t* sels)
{
    const Bsr& b = l.b;
    int first = 0;
    for (int seg = 0; seg < l.nseg; ++seg) {
        const int rows = l.rows_of(seg);
        const uint32_t* const m = &l.masks[(size_t)(t * l.K + (int64_t)seg * SEGMENT_ROWS)];
        for (int s = 0; s < segments[seg].steps; ++s) {
            uint8_t* const r = rec + (int64_t)(first + s) * WIDE_RECORD_BYTES;
            std::memset(r, 0, WIDE_VAL_BYTES);
            const int32_t* const slot = segments[seg].slot + s * STEP_K;
            for (int q = 0; q < STEP_K / 4; ++q) {
                uint32_t before = 0;
                for (int z = 4 * q; z < 4 * q + 4; ++z) {
                    const int k = slot[z], pad = ((z & 7) + (z >> 3)) & 7;
                    set_row(r, z, k >= 0 ? k : pad < rows ? pad : 0);
                    if (k < 0) continue;
                    const int h = z >> 4 & 1, which = 8 * (z >> 5) + 2 * (z >> 2 & 3);
                    places[(size_t)(seg * SEGMENT_ROWS + k)] = {(uint32_t)((first + s) * WIDE_RECORD_BYTES + 32 * h * 16 + which), before,
                                                               (uint16_t)(2 * (first + s) + h), (uint8_t)(z & 3), (uint8_t)(2 * which)};
                    before |= m[k];
                }
            }
        }
        first += segments[seg].steps;
    }
    const int units = l.units, rows_of_unit = WIDE_ROWS / units;
    std::memset(sels, 0, (size_t)(2 * first * units) * 4);
    auto add = [&](const WidePlace& p, const int u, const int row, const int rows, const uint32_t v) {
        const uint32_t second = p.before >> u & 1;
        uint8_t* const to = rec + p.at + second + 16 * row;
        for (int i = 0; i < rows; ++i) to[16 * i] = (uint8_t)(v >> (8 * i));
        sels[(size_t)(p.sel_word * units + u)] |= (uint32_t)p.sel << (p.shift + 2 * second);
    };
    for (int u = 0; u < units && t * units + u < b.block_rows; ++u) {
        const int64_t br = t * units + u;
        for (int64_t e = b.row_ptr[(size_t)br]; e < b.row_ptr[(size_t)br + 1]; ++e) {
            uint32_t v;
            std::memcpy(&v, &b.vals[(size_t)e * 4], 4);
            const int64_t k = b.index[(size_t)e];
            if (l.n4) {
                add(places[(size_t)k], u, 4 * u, 4, v);
            } else {
                for (int j = 0; j < 4; ++j)
                    if (v >> (8 * j) & 0xff) add(places[(size_t)(4 * k + j)], u, u, 1, v >> (8 * j) & 0xff);
            }
        }
    }
    for (int s = 0; s < first; ++s) {
        uint8_t* const to = rec + (int64_t)s * WIDE_RECORD_BYTES + WIDE_VAL_BYTES;
        for (int h = 0; h < 2; ++h)
            for (int row = 0; row < WIDE_ROWS; ++row) std::memcpy(to + 8 * (32 * h + row), &sels[(size_t)((2 * s + h) * units + row / rows_of_unit)], 4);
    }
    std::memset(rec + (int64_t)first * WIDE_RECORD_BYTES, 0, (size_t)((room - first) * WIDE_RECORD_BYTES));
}

// what the steps of every (wide tile, segment) come to
struct WideDims {
    std::vector<int64_t> first;     // record of every tile
    int64_t records = 0;
    WideDims(int nseg, int64_t nt, const int32_t* steps, DeviceForms& f) : first((size_t)nt + 1, 0)
    {
        f.wide_max_steps = 0;
        int most = 0;
        for (int64_t t = 0; t < nt; ++t) {
            int all = 0;
            for (int seg = 0; seg < nseg; ++seg) {
                all += steps[(size_t)(t * nseg + seg)];
                f.wide_max_steps = std::max(f.wide_max_steps, steps[(size_t)(t * nseg + seg)]);
            }
            most = std::max(most, all);
            first[(size_t)t + 1] = first[(size_t)t] + all;
        }
        f.wide_max_steps = std::max(1, f.wide_max_steps);
        f.wide_nsteps = first.back();
        f.wide_tile_steps = nt * most <= f.wide_nsteps + f.wide_nsteps / 2 ? most : 0;
        if (f.wide_tile_steps)
            for (int64_t t = 0; t <= nt; ++t) first[(size_t)t] = t * most;
        records = std::max<int64_t>(1, first.back());
        f.wide_size = wide_records_offset(nt, nseg) + records * WIDE_RECORD_BYTES;
    }
};

// and those of the row tiles
void narrow_dims(const HostLayout& hl, DeviceForms& f)
{
    f.tile_steps = (int64_t)hl.ntiles * hl.max_steps_per_tile <= hl.nsteps + hl.nsteps / 2 ? hl.max_steps_per_tile : 0;
    const int64_t records = std::max<int64_t>(1, f.tile_steps ? (int64_t)hl.ntiles * f.tile_steps : hl.nsteps);
    f.size = (records_offset(hl.ntiles, hl.nseg) + records * RECORD_BYTES + 127) & ~(int64_t)127;
}

}  // namespace

void forms_from_bsr(const Bsr& b, HostLayout& hl, DeviceForms& f, Team& team, const std::function<void()>& first_form)
{
    hl.rowsum.assign((size_t)((b.N + TILE_ROWS - 1) / TILE_ROWS) * TILE_ROWS, 0);
    Lists l(b, hl.rowsum.data(), team);
    layout_dims(l.nseg, l.ntiles, l.steps.data(), hl);
    const int64_t nt16 = l.ntiles, ns = l.nseg;
    narrow_dims(hl, f);
    WideDims dims(l.nseg, l.nt, l.wide_steps.data(), f);
    f.together = f.size + f.wide_size <= 256 * 1024;
    f.bytes.reset(new uint8_t[(size_t)(f.size + (f.together ? f.wide_size : 0))]);
    // The wide form is not needed to run the weight: without memory for it there is none.
    std::atomic<bool> none{false}, longer{false};
    auto wide_memory = [&](const auto& get) {
        try {
            get();
        } catch (const std::bad_alloc&) {
            none = true;
        }
    };
    if (!f.together) wide_memory([&] { f.wide.reset(new uint8_t[(size_t)f.wide_size]); });

    auto narrow_tile = [&](int64_t t, int32_t* place) {
        uint8_t* const rec = f.bytes.get() + records_offset(nt16, ns);
        int32_t* const bounds = (int32_t*)(f.bytes.get() + bounds_offset(nt16)) + t * (ns + 1);
        const int64_t first = hl.seg_ptr[(size_t)(t * ns)], at = f.tile_steps ? t * f.tile_steps : first;
        for (int64_t g = 0; g <= ns; ++g) bounds[g] = (int32_t)(hl.seg_ptr[(size_t)(t * ns + g)] - first + at);
        uint8_t* const to = rec + at * RECORD_BYTES;
        arrange_tile(l, t, to, RECORD_BYTES, to + STEP_VAL_BYTES, RECORD_BYTES, true, place);
        const int64_t used = hl.seg_ptr[(size_t)((t + 1) * ns)] - first, room = f.tile_steps ? f.tile_steps : used;
        std::memset(to + used * RECORD_BYTES, 0, (size_t)((room - used) * RECORD_BYTES));
    };
    team.run(nt16, 2 * l.grain, [&](int64_t begin, int64_t end) {
        const std::unique_ptr<int32_t[]> place(new int32_t[(size_t)l.K]);
        for (int64_t t = begin; t < end; ++t) narrow_tile(t, place.get());
    });
    // row sums, and what is between the bounds and the records
    const size_t sums = hl.rowsum.size() * 4, narrow_end = (size_t)(bounds_offset(nt16) + nt16 * (ns + 1) * 4);
    std::memcpy(f.bytes.get(), hl.rowsum.data(), sums);
    std::memset(f.bytes.get() + narrow_end, 0, (size_t)records_offset(nt16, ns) - narrow_end);
    if (!hl.nsteps) std::memset(f.bytes.get() + records_offset(nt16, ns), 0, RECORD_BYTES);

    // Every tile is packed where it goes if no list needs more steps than its length asks for.  Those that do are kept as they
    // are arranged, for a second pass.  (256x256 in 1x4 blocks at 70 %, where all do, on the host: 0.38 ms; 1.0 when the second
    // pass arranged all tiles anew, slot by slot; 0.30 for the first form alone.)
    std::vector<std::unique_ptr<WideSegment[]>> kept;
    wide_memory([&] { kept.resize((size_t)l.nt); });
    auto wide_tiles = [&](int64_t begin, int64_t end, const auto& tile) {
        std::unique_ptr<WidePlace[]> places;
        std::unique_ptr<uint32_t[]> sels;
        wide_memory([&] {
            places.reset(new WidePlace[(size_t)l.K]);
            sels.reset(new uint32_t[(size_t)(2 * ns * WIDE_MAX_STEPS * l.units)]);
        });
        uint8_t* const form = f.wide_bytes();
        for (int64_t t = begin; t < end && !none; ++t) {
            const int64_t first = dims.first[(size_t)t], room = dims.first[(size_t)t + 1] - first;
            uint8_t* const rec = form + wide_records_offset(l.nt, ns) + first * WIDE_RECORD_BYTES;
            if (const WideSegment* const segments = tile(t, rec, room)) write_wide_tile(l, t, segments, rec, room, places.get(), sels.get());
            int32_t* const bounds = (int32_t*)(form + wide_bounds_offset(l.nt)) + t * (ns + 1);
            bounds[0] = (int32_t)first;
            for (int64_t g = 0; g < ns; ++g) bounds[g + 1] = bounds[g] + l.wide_steps[(size_t)(t * ns + g)];
        }
    };
    team.finish(l.nt, l.grain, [&](int64_t begin, int64_t end) {
        std::unique_ptr<WideSegment[]> segments;
        wide_tiles(begin, end, [&](int64_t t, uint8_t*, int64_t) -> const WideSegment* {
            bool more = false;
            wide_memory([&] {
                if (!segments) segments.reset(new WideSegment[(size_t)ns]);
            });
            if (none || !arrange_segments(l, t, segments.get(), &l.wide_steps[(size_t)(t * ns)], more)) {
                none = true;
                return nullptr;
            }
            if (!more) return segments.get();
            longer = true;
            kept[(size_t)t] = std::move(segments);
            return nullptr;
        });
    }, first_form);
    // (lists that two of a quad lengthen, 1x4 blocks at 75 % for instance: the tiles to where they go now that all steps are known)
    if (longer && !none) {
        const std::vector<int64_t> was_at = dims.first;
        const std::unique_ptr<uint8_t[]> old = std::move(f.wide);
        const uint8_t* const from = f.together ? f.bytes.get() + f.size : old.get();
        dims = WideDims(l.nseg, l.nt, l.wide_steps.data(), f);
        wide_memory([&] { f.wide.reset(new uint8_t[(size_t)f.wide_size]); });
        f.together = false;
        Team again;
        again.finish(l.nt, l.grain, [&](int64_t begin, int64_t end) {
            wide_tiles(begin, end, [&](int64_t t, uint8_t* rec, int64_t room) -> const WideSegment* {
                if (kept[(size_t)t]) return kept[(size_t)t].get();
                const int64_t records = was_at[(size_t)t + 1] - was_at[(size_t)t];
                std::memcpy(rec, from + wide_records_offset(l.nt, ns) + was_at[(size_t)t] * WIDE_RECORD_BYTES, (size_t)(records * WIDE_RECORD_BYTES));
                std::memset(rec + records * WIDE_RECORD_BYTES, 0, (size_t)((room - records) * WIDE_RECORD_BYTES));
                return nullptr;
            });
        });
    }
    if (none) {
        f.drop_wide();
        return;
    }
    uint8_t* const form = f.wide_bytes();
    const size_t wide_end = (size_t)(wide_bounds_offset(l.nt) + l.nt * (ns + 1) * 4);
    std::memcpy(form, hl.rowsum.data(), sums);
    std::memset(form + sums, 0, (size_t)wide_bounds_offset(l.nt) - sums);
    std::memset(form + wide_end, 0, (size_t)wide_records_offset(l.nt, ns) - wide_end);
    if (!f.wide_nsteps) std::memset(form + wide_records_offset(l.nt, ns), 0, WIDE_RECORD_BYTES);
}

void dims_from_steps(int64_t N, int64_t K, const int32_t* steps, const int32_t* wide_steps, const int32_t* sums, HostLayout& hl,
                     DeviceForms& f, std::vector<uint8_t>& heads, int64_t& head)
{
    const int64_t ns = (K + SEGMENT_ROWS - 1) / SEGMENT_ROWS, nt16 = (N + TILE_ROWS - 1) / TILE_ROWS, nt = (nt16 + 1) / 2;
    hl.rowsum.assign((size_t)(nt16 * TILE_ROWS), 0);
    for (int64_t t = 0; t < nt; ++t)
        for (int64_t g = 0; g < ns; ++g)
            for (int64_t r = t * WIDE_ROWS; r < std::min((t + 1) * WIDE_ROWS, nt16 * TILE_ROWS); ++r)
                hl.rowsum[(size_t)r] += sums[(t * ns + g) * WIDE_ROWS + r - t * WIDE_ROWS];
    layout_dims((int)ns, (int)nt16, steps, hl);
    narrow_dims(hl, f);
    head = records_offset(nt16, ns) + (hl.nsteps ? 0 : RECORD_BYTES);
    heads.assign((size_t)head, 0);
    const size_t rowsums = hl.rowsum.size() * 4;
    std::memcpy(heads.data(), hl.rowsum.data(), rowsums);
    int32_t* bounds = (int32_t*)(heads.data() + bounds_offset(nt16));
    for (int64_t t = 0; t < nt16; ++t) {
        const int64_t first = hl.seg_ptr[(size_t)(t * ns)], at = f.tile_steps ? t * f.tile_steps : first;
        for (int64_t g = 0; g <= ns; ++g) *bounds++ = (int32_t)(hl.seg_ptr[(size_t)(t * ns + g)] - first + at);
    }
    f.together = false;
    if (std::any_of(wide_steps, wide_steps + nt * ns, [](int32_t s) { return s < 0; })) {
        f.drop_wide();
        return;
    }
    const WideDims dims((int)ns, nt, wide_steps, f);
    heads.resize((size_t)(head + wide_records_offset(nt, ns) + (f.wide_nsteps ? 0 : WIDE_RECORD_BYTES)), 0);
    std::memcpy(heads.data() + head, hl.rowsum.data(), rowsums);
    bounds = (int32_t*)(heads.data() + head + wide_bounds_offset(nt));
    for (int64_t t = 0; t < nt; ++t) {
        *bounds = (int32_t)dims.first[(size_t)t];
        for (int64_t g = 0; g < ns; ++g, ++bounds) bounds[1] = bounds[0] + wide_steps[t * ns + g];
        ++bounds;
    }
}

}  // namespace spmm
