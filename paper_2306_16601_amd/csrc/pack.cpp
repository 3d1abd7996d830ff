// Host-side packer: dense-with-zeros int8 weight -> canonical 4x1 block-sparse rows ->
// the device's row-tile union layout (see spmm_internal.h).  Pure C++, no GPU calls.
//
// Paper Section 3.1 / Figure 1: blocks of 4x1 with the sparsity dimension on the output
// channels.  Section 3.2: the kernel is specialised on the sparse weight and its indices,
// and the block count is padded to what the multiply instruction accumulates over (note
// after Algorithm 1).  Here that instruction is the 16x16x64 int8 matrix op, so the unit
// of padding is 64 listed k positions per 16-row tile.
#include <algorithm>
#include <atomic>
#include <cstring>
#include <exception>
#include <memory>
#include <thread>

#include "spmm_internal.h"

namespace spmm {

namespace {

// f(begin, end) over [0, n) in at most 8 threads, each with at least `grain` items; the first exception of a
// thread is rethrown here.  (Packing a model's weights is what its load waits for; row tiles are independent.)
template <typename F>
void parallel_for(int64_t n, int64_t grain, const F& f)
{
    const int64_t hw = std::max<int64_t>(1, std::thread::hardware_concurrency());
    const int64_t parts = std::max<int64_t>(1, std::min<int64_t>({8, hw, n / std::max<int64_t>(1, grain)}));
    if (parts == 1) {
        f((int64_t)0, n);
        return;
    }
    std::vector<std::exception_ptr> failed((size_t)parts);
    std::vector<std::thread> threads;
    threads.reserve((size_t)parts - 1);
    auto part = [&](int64_t i) {
        try {
            f(n * i / parts, n * (i + 1) / parts);
        } catch (...) {
            failed[(size_t)i] = std::current_exception();
        }
    };
    int64_t started = 1;
    try {
        for (; started < parts; ++started) threads.emplace_back(part, started);
    } catch (...) {      // no more threads to be had: the rest of the work is done here
    }
    part(0);
    for (int64_t i = started; i < parts; ++i) part(i);
    for (std::thread& t : threads) t.join();
    for (const std::exception_ptr& e : failed)
        if (e) std::rethrow_exception(e);
}

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

// The blocks of block-row br, at most K of them, to index / vals (4 bytes per block, as one dword); returns how many
int64_t blocks_of_row(const int8_t* W, int64_t N, int64_t K, int64_t ldw, spmm_block_t block, int64_t br, int32_t* index,
                      uint32_t* vals)
{
    int64_t n = 0;
    if (block == SPMM_BLOCK_N4K1) {
        const int rows = (int)std::min<int64_t>(4, N - br * 4);
        const int8_t* r[4];
        for (int i = 0; i < 4; ++i) r[i] = W + (br * 4 + std::min(i, rows - 1)) * ldw;     // (missing rows: the last one again)
        const uint32_t keep = rows == 4 ? 0xffffffffu : (1u << (8 * rows)) - 1u;
        auto add = [&](int64_t k) {
            index[n] = (int32_t)k;
            vals[n++] = ((uint32_t)(uint8_t)r[0][k] | (uint32_t)(uint8_t)r[1][k] << 8 | (uint32_t)(uint8_t)r[2][k] << 16 |
                         (uint32_t)(uint8_t)r[3][k] << 24) & keep;
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
        for (int64_t c = 0; c * 4 < K; ++c) {
            uint32_t v = 0;
            std::memcpy(&v, r + 4 * c, (size_t)std::min<int64_t>(4, K - 4 * c));
            if (v) {
                index[n] = (int32_t)c;
                vals[n++] = v;
            }
        }
    }
    return n;
}

}  // namespace

void bsr_from_dense(const int8_t* W, int64_t N, int64_t K, int64_t ldw, spmm_block_t block, Bsr& out)
{
    out.N = N;
    out.K = K;
    out.block = block;
    out.block_rows = (block == SPMM_BLOCK_N4K1) ? (N + 3) / 4 : N;
    out.row_ptr.assign((size_t)out.block_rows + 1, 0);
    // every thread collects its block-rows, then the pieces are put together
    struct Piece { int64_t first; std::vector<int32_t> index; std::vector<uint32_t> vals; };
    std::vector<Piece> pieces(8);
    std::atomic<int> used{0};
    const int64_t rows_per_block_row = (block == SPMM_BLOCK_N4K1) ? 4 : 1;
    parallel_for(out.block_rows, std::max<int64_t>(1, 131072 / (K * rows_per_block_row)), [&](int64_t begin, int64_t end) {
        Piece& p = pieces[(size_t)used.fetch_add(1)];
        p.first = begin;
        p.index.reserve((size_t)((end - begin) * K / 3));
        p.vals.reserve((size_t)((end - begin) * K / 3));
        std::vector<int32_t> index((size_t)K);
        std::vector<uint32_t> vals((size_t)K);
        for (int64_t br = begin; br < end; ++br) {
            const int64_t n = blocks_of_row(W, N, K, ldw, block, br, index.data(), vals.data());
            p.index.insert(p.index.end(), index.begin(), index.begin() + n);
            p.vals.insert(p.vals.end(), vals.begin(), vals.begin() + n);
            out.row_ptr[(size_t)br + 1] = (int64_t)p.index.size();      // within the piece, for now
        }
    });
    pieces.resize((size_t)used.load());
    std::sort(pieces.begin(), pieces.end(), [](const Piece& x, const Piece& y) { return x.first < y.first; });
    int64_t total = 0;
    for (size_t i = 0; i < pieces.size(); ++i) {
        const int64_t end = i + 1 < pieces.size() ? pieces[i + 1].first : out.block_rows;
        for (int64_t br = pieces[i].first; br < end; ++br) out.row_ptr[(size_t)br + 1] += total;
        total += (int64_t)pieces[i].index.size();
    }
    out.index.resize((size_t)total);
    out.vals.resize((size_t)total * 4);
    int64_t at = 0;
    for (const Piece& p : pieces) {
        if (p.index.empty()) continue;
        std::memcpy(&out.index[(size_t)at], p.index.data(), p.index.size() * sizeof(int32_t));
        std::memcpy(&out.vals[(size_t)at * 4], p.vals.data(), p.vals.size() * 4);
        at += (int64_t)p.index.size();
    }
}

void bsr_to_dense(const Bsr& b, int8_t* W, int64_t ldw)
{
    const bool n4 = b.block == SPMM_BLOCK_N4K1;
    parallel_for(b.block_rows, std::max<int64_t>(1, 262144 / (b.K * (n4 ? 4 : 1))), [&](int64_t begin, int64_t end) {
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
// slot_k[s*64 + 16*g + t] = segment-local k or -1 (padding); slot_row = row actually read.
static void arrange_for_lds_banks(const int32_t* list, int n_listed, int rows_in_segment, int nsteps, int32_t* slot_k,
                                  int32_t* slot_row)
{
    constexpr int MAXH = 4 * SEGMENT_ROWS / STEP_K;     // half-reads of the longest list
    const int H = 4 * nsteps;
    if (nsteps == 0) return;
    // entries by residue
    int32_t by_res[16][SEGMENT_ROWS / 16];
    int n_res[16] = {0};
    for (int i = 0; i < n_listed; ++i) by_res[list[i] & 15][n_res[list[i] & 15]++] = list[i];
    int order[16];
    for (int r = 0; r < 16; ++r) order[r] = r;
    std::stable_sort(order, order + 16, [&](int x, int y) { return n_res[x] > n_res[y]; });

    // Largest residue class first; each class is spread over the least-filled half-reads, one
    // entry per half-read, so that no half-read runs out of room while others still have
    // holes.  Only a class with more than H entries is forced to double up somewhere.
    int32_t hr[MAXH][16];
    int load[MAXH] = {0}, by_load[MAXH];
    uint32_t mask[MAXH] = {0};
    for (int oi = 0; oi < 16; ++oi) {
        const int r = order[oi];
        int next = 0;
        while (next < n_res[r]) {
            int count[18] = {0};                        // half-reads by load (at most 16), stable
            for (int h = 0; h < H; ++h) ++count[load[h] + 1];
            for (int l = 1; l < 18; ++l) count[l] += count[l - 1];
            for (int h = 0; h < H; ++h) by_load[count[load[h]]++] = h;
            bool placed = false;
            for (int i = 0; i < H && next < n_res[r]; ++i) {
                const int h = by_load[i];
                if (load[h] >= 16) break;
                hr[h][load[h]++] = by_res[r][next++];
                mask[h] |= 1u << r;
                placed = true;
            }
            if (!placed) break;   // cannot happen: 16 * H slots >= n_listed
        }
    }
    for (int h = 0; h < H; ++h) {
        const int s = h / 4, instr = (h / 2) % 2, pair = h % 2;
        int next_res = 0;
        for (int j = 0; j < 16; ++j) {
            const int g = 2 * pair + j / 8, t = 8 * instr + j % 8;
            const int slot = s * STEP_K + 16 * g + t;
            if (j < load[h]) {
                slot_k[slot] = hr[h][j];
                slot_row[slot] = hr[h][j];
            } else {
                while (next_res < 16 && (mask[h] & (1u << next_res))) ++next_res;
                int row = 0;
                if (next_res < 16) {
                    if (next_res < rows_in_segment) row = next_res;
                    mask[h] |= 1u << next_res;
                }
                slot_k[slot] = -1;
                slot_row[slot] = row;
            }
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

void layout_from_bsr(const Bsr& b, int kc, HostLayout& out)
{
    const int64_t N = b.N, K = b.K;
    const bool n4 = b.block == SPMM_BLOCK_N4K1;
    out.kc = kc;                                            // SEGMENT_ROWS
    out.nseg = (int)((K + kc - 1) / kc);
    out.ntiles = (int)((N + TILE_ROWS - 1) / TILE_ROWS);
    out.rowsum.assign((size_t)out.ntiles * TILE_ROWS, 0);
    out.max_steps_per_tile = 0;
    out.max_steps_per_segment = 0;
    const int nseg = out.nseg, seg_words = kc / 64;
    const int units = n4 ? TILE_ROWS / 4 : TILE_ROWS;       // block-rows of a tile
    const int64_t grain = std::max<int64_t>(1, 262144 / (K * TILE_ROWS));

    // ---- the union of every tile's k lists, one bit per k; rows past N and block-rows past the end have none
    std::vector<uint64_t> listed((size_t)out.ntiles * nseg * seg_words, 0);
    std::vector<int32_t> steps((size_t)out.ntiles * nseg);
    parallel_for(out.ntiles, grain, [&](int64_t begin, int64_t end) {
        for (int64_t tile = begin; tile < end; ++tile) {
            uint64_t* const bits = &listed[(size_t)(tile * nseg) * seg_words];
            int32_t* const sum = &out.rowsum[(size_t)tile * TILE_ROWS];
            for (int q = 0; q < units && tile * units + q < b.block_rows; ++q) {
                const int64_t br = tile * units + q;
                for (int64_t e = b.row_ptr[(size_t)br]; e < b.row_ptr[(size_t)br + 1]; ++e) {
                    const int8_t* v = &b.vals[(size_t)e * 4];
                    if (n4) {
                        const int32_t k = b.index[(size_t)e];
                        bits[k >> 6] |= (uint64_t)1 << (k & 63);
                        for (int i = 0; i < 4; ++i) sum[4 * q + i] += v[i];
                    } else {
                        for (int j = 0; j < 4; ++j) {
                            const int32_t k = b.index[(size_t)e] * 4 + j;
                            if (v[j]) bits[k >> 6] |= (uint64_t)1 << (k & 63);
                            sum[q] += v[j];
                        }
                    }
                }
            }
            for (int seg = 0; seg < nseg; ++seg) {
                int n = 0;
                for (int w = 0; w < seg_words; ++w) n += __builtin_popcountll(bits[seg * seg_words + w]);
                steps[(size_t)(tile * nseg + seg)] = (n + STEP_K - 1) / STEP_K;
            }
        }
    });
    out.seg_ptr.assign((size_t)out.ntiles * nseg + 1, 0);
    for (int64_t tile = 0; tile < out.ntiles; ++tile) {
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
    out.vals.assign((size_t)out.nsteps * STEP_VAL_BYTES, 0);
    out.idx.assign((size_t)out.nsteps * STEP_IDX_DWORDS, 0);

    // ---- the steps: listed k dealt to slots, every block's values scattered to their lanes
    parallel_for(out.ntiles, grain, [&](int64_t begin, int64_t end) {
        std::vector<int32_t> place((size_t)K);              // k -> 64 * step + slot, for the k listed in this tile
        int32_t list[SEGMENT_ROWS], slot_k[SEGMENT_ROWS], slot_row[SEGMENT_ROWS];
        for (int64_t tile = begin; tile < end; ++tile) {
            for (int seg = 0; seg < nseg; ++seg) {
                const size_t i = (size_t)(tile * nseg + seg);
                const int k_lo = seg * kc, rows = (int)std::min<int64_t>(kc, K - k_lo);
                int n = 0;
                for (int w = 0; w < seg_words; ++w)
                    for (uint64_t m = listed[i * seg_words + w]; m; m &= m - 1) list[n++] = 64 * w + __builtin_ctzll(m);
                arrange_for_lds_banks(list, n, rows, steps[i], slot_k, slot_row);
                for (int s = 0; s < steps[i]; ++s) {
                    const int32_t* sk = slot_k + s * STEP_K;     // segment-local k, -1 = padding
                    const int32_t* sr = slot_row + s * STEP_K;   // activation row the slot reads
                    const int32_t step = out.seg_ptr[i] + s;
                    for (int t = 0; t < STEP_K; ++t)
                        if (sk[t] >= 0) place[(size_t)(k_lo + sk[t])] = (s + out.seg_ptr[i] - out.seg_ptr[(size_t)(tile * nseg)]) * STEP_K + t;
                    uint32_t* const ix = &out.idx[(size_t)step * STEP_IDX_DWORDS];
                    for (int g = 0; g < 4; ++g)
                        for (int t = 0; t < 8; ++t) ix[8 * g + t] = (uint32_t)sr[16 * g + t] | ((uint32_t)sr[16 * g + 8 + t] << 16);
                }
            }
            if (out.seg_ptr[(size_t)(tile * nseg)] == out.seg_ptr[(size_t)((tile + 1) * nseg)]) continue;
            // vals[step][lane = 16 g + row][t] of slot 16 g + t
            uint8_t* const vals = &out.vals[(size_t)out.seg_ptr[(size_t)(tile * nseg)] * STEP_VAL_BYTES];
            auto lane_bytes = [&](int32_t k) {              // of row 0; row r is 16 r bytes on
                const int32_t p = place[(size_t)k], slot = p & (STEP_K - 1);
                return vals + (size_t)(p / STEP_K) * STEP_VAL_BYTES + (size_t)(slot & ~15) * 16 + (slot & 15);
            };
            for (int q = 0; q < units && tile * units + q < b.block_rows; ++q) {
                const int64_t br = tile * units + q;
                for (int64_t e = b.row_ptr[(size_t)br]; e < b.row_ptr[(size_t)br + 1]; ++e) {
                    uint32_t v;
                    std::memcpy(&v, &b.vals[(size_t)e * 4], 4);
                    const int32_t at = b.index[(size_t)e];
                    if (n4) {
                        uint8_t* const to = lane_bytes(at) + 4 * q * 16;
                        for (int j = 0; j < 4; ++j) to[16 * j] = (uint8_t)(v >> (8 * j));
                    } else {
                        for (int j = 0; j < 4; ++j)
                            if (v >> (8 * j) & 0xff) *(lane_bytes(at * 4 + j) + q * 16) = (uint8_t)(v >> (8 * j));
                    }
                }
            }
        }
    });
}

void device_form(const HostLayout& hl, int tile_steps, int64_t records, uint8_t* out)
{
    const int64_t nt = hl.ntiles, ns = hl.nseg, at = records_offset(nt, ns);
    std::memset(out, 0, (size_t)at);
    std::memcpy(out, hl.rowsum.data(), hl.rowsum.size() * 4);
    int32_t* const bounds = (int32_t*)(out + bounds_offset(nt));
    uint8_t* const rec = out + at;
    if (nt * tile_steps == 0 && hl.nsteps == 0) std::memset(rec, 0, (size_t)records * RECORD_BYTES);
    parallel_for(nt, std::max<int64_t>(1, 262144 / std::max<int64_t>(1, records * RECORD_BYTES / nt)), [&](int64_t begin, int64_t end) {
        for (int64_t t = begin; t < end; ++t) {
            const int64_t first = hl.seg_ptr[(size_t)(t * ns)], past = hl.seg_ptr[(size_t)((t + 1) * ns)];
            const int64_t shift = tile_steps ? t * tile_steps - first : 0;
            for (int64_t g = 0; g <= ns; ++g) bounds[t * (ns + 1) + g] = (int32_t)(hl.seg_ptr[(size_t)(t * ns + g)] + shift);
            for (int64_t g = 0; g < ns; ++g) {
                const uint32_t base = (uint32_t)(g * SEGMENT_ROWS) * 0x10001u;      // the rows of the whole weight
                for (int64_t s = hl.seg_ptr[(size_t)(t * ns + g)]; s < hl.seg_ptr[(size_t)(t * ns + g + 1)]; ++s) {
                    uint8_t* const r = rec + (s + shift) * RECORD_BYTES;
                    std::memcpy(r, &hl.vals[(size_t)s * STEP_VAL_BYTES], STEP_VAL_BYTES);
                    for (int i = 0; i < STEP_IDX_DWORDS; ++i) {
                        const uint32_t v = hl.idx[(size_t)s * STEP_IDX_DWORDS + i] + base;
                        std::memcpy(r + STEP_VAL_BYTES + 4 * i, &v, 4);
                    }
                }
            }
            if (tile_steps) std::memset(rec + (past + shift) * RECORD_BYTES, 0, (size_t)(tile_steps - (past - first)) * RECORD_BYTES);
        }
    });
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

struct WideSegment {
    int32_t slot[WIDE_MAX_STEPS * STEP_K];      // segment-local k, -1: padding
    int steps;
};

// false: more than WIDE_MAX_STEPS
bool arrange_wide(const uint32_t* mask, int rows, WideSegment& out)
{
    constexpr int CLASSES = 8, MAX_QUADS = WIDE_MAX_STEPS * STEP_K / 4;
    // candidates of every class, heaviest first, and for every unit which of them it uses
    int32_t cand[CLASSES][SEGMENT_ROWS / CLASSES];
    uint64_t alive[CLASSES], uses[CLASSES][32];
    std::memset(uses, 0, sizeof(uses));
    int n = 0;
    for (int c = 0; c < CLASSES; ++c) {
        uint8_t weight[SEGMENT_ROWS / CLASSES];
        int start[34] = {0}, m = 0;
        for (int k = c, i = 0; k < rows; k += CLASSES, ++i) {
            weight[i] = (uint8_t)__builtin_popcount(mask[k]);
            if (weight[i]) { ++start[32 - weight[i] + 1]; ++m; }
        }
        for (int w = 1; w < 34; ++w) start[w] += start[w - 1];
        for (int k = c, i = 0; k < rows; k += CLASSES, ++i) {
            if (!weight[i]) continue;
            const int at = start[32 - weight[i]]++;
            cand[c][at] = k;
            for (uint32_t u = mask[k]; u; u &= u - 1) uses[c][__builtin_ctz(u)] |= (uint64_t)1 << at;
        }
        alive[c] = m == 64 ? ~(uint64_t)0 : ((uint64_t)1 << m) - 1;
        n += m;
    }
    out.steps = (n + STEP_K - 1) / STEP_K;
    uint32_t one[MAX_QUADS] = {0}, two[MAX_QUADS] = {0};       // units with a k, with two, in the quad
    auto put = [&](int slot, int32_t k) {
        out.slot[slot] = k;
        two[slot / 4] |= one[slot / 4] & mask[k];
        one[slot / 4] |= mask[k];
    };
    for (int i = 0; i < out.steps * STEP_K; ++i) out.slot[i] = -1;
    for (int o = 0; o < out.steps * 8; ++o) {
        for (int j = 0; j < 8; ++j) {
            const int c = (j + o) & 7;
            uint64_t fit = alive[c];
            for (uint32_t u = two[2 * o + j / 4]; u; u &= u - 1) fit &= ~uses[c][__builtin_ctz(u)];
            if (!fit) continue;
            alive[c] &= ~(fit & (0 - fit));
            put(8 * o + j, cand[c][__builtin_ctzll(fit)]);
        }
    }
    // what is left over
    int exchanges = 256;                            // (a bound on the work; then a new step)
    for (int c = 0; c < CLASSES; ++c) {
        while (alive[c]) {
            const int32_t k = cand[c][__builtin_ctzll(alive[c])];
            const uint32_t m = mask[k];
            bool done = false;
            auto hole_of = [&](int q) {
                for (int s = 4 * q; s < 4 * q + 4; ++s)
                    if (out.slot[s] < 0) return s;
                return -1;
            };
            int holes[MAX_QUADS], nholes = 0;
            for (int q = 0; q < out.steps * 16; ++q)
                if (hole_of(q) >= 0) holes[nholes++] = q;
            for (int i = 0; i < nholes && !done; ++i)
                if (!(two[holes[i]] & m)) {
                    put(hole_of(holes[i]), k);
                    done = true;
                }
            // a k of another quad into the hole, and this one into its place
            for (int i = 0; i < nholes && !done && exchanges-- > 0; ++i) {
                const int q = holes[i];
                for (int s = 0; s < out.steps * STEP_K && !done; ++s) {
                    const int r = s / 4;
                    if (r == q || out.slot[s] < 0 || (two[q] & mask[out.slot[s]])) continue;
                    uint32_t o1 = 0, t1 = 0;        // quad r without slot s
                    for (int z = 4 * r; z < 4 * r + 4; ++z)
                        if (z != s && out.slot[z] >= 0) {
                            t1 |= o1 & mask[out.slot[z]];
                            o1 |= mask[out.slot[z]];
                        }
                    if (t1 & m) continue;
                    put(hole_of(q), out.slot[s]);
                    one[r] = o1;
                    two[r] = t1;
                    put(s, k);
                    done = true;
                }
            }
            if (!done) {
                if (out.steps == WIDE_MAX_STEPS) return false;
                for (int i = 0; i < STEP_K; ++i) out.slot[out.steps * STEP_K + i] = -1;
                ++out.steps;
                continue;                           // (and again, now that there are holes)
            }
            alive[c] &= alive[c] - 1;
        }
    }
    return true;
}

}  // namespace

// activation row of slot z of a record, at the lanes that gather it
static void set_row(uint8_t* record, int z, int row)
{
    uint16_t* const r = (uint16_t*)(record + WIDE_VAL_BYTES);
    const int lane = 32 * (z >> 5) + 2 * (z & 7) + (z >> 4 & 1), half = z >> 3 & 1;
    r[4 * lane + 2 + half] = r[4 * (lane + 16) + 2 + half] = (uint16_t)(32 * row);
}

bool wide_from_bsr(const Bsr& b, WideForm& out)
{
    const int64_t N = b.N, K = b.K;
    const bool n4 = b.block == SPMM_BLOCK_N4K1;
    const int units = n4 ? WIDE_ROWS / 4 : WIDE_ROWS;
    out.nseg = (int)((K + SEGMENT_ROWS - 1) / SEGMENT_ROWS);
    out.ntiles = (int)((N + WIDE_ROWS - 1) / WIDE_ROWS);
    const int nseg = out.nseg;
    const int64_t nt = out.ntiles, grain = std::max<int64_t>(1, 262144 / (K * WIDE_ROWS));
    std::vector<int32_t> steps((size_t)(nt * nseg));
    // of every k listed in a tile: 64 * step + slot, and the units that have a k in an earlier slot of its quad
    struct Place { int32_t slot; uint32_t before; };
    std::unique_ptr<Place[]> places(new Place[(size_t)(nt * K)]);
    std::atomic<bool> fits{true};
    parallel_for(nt, grain, [&](int64_t begin, int64_t end) {
        std::vector<uint32_t> mask((size_t)K);
        WideSegment seg_slots;
        for (int64_t t = begin; t < end && fits; ++t) {
            std::fill(mask.begin(), mask.end(), 0u);
            for (int u = 0; u < units && t * units + u < b.block_rows; ++u) {
                const int64_t br = t * units + u;
                for (int64_t e = b.row_ptr[(size_t)br]; e < b.row_ptr[(size_t)br + 1]; ++e) {
                    if (n4) {
                        mask[(size_t)b.index[(size_t)e]] |= 1u << u;
                    } else {
                        for (int j = 0; j < 4; ++j)
                            if (b.vals[(size_t)e * 4 + j]) mask[(size_t)b.index[(size_t)e] * 4 + j] |= 1u << u;
                    }
                }
            }
            int first = 0;
            for (int seg = 0; seg < nseg; ++seg) {
                const int64_t k0 = (int64_t)seg * SEGMENT_ROWS;
                const int rows = (int)std::min<int64_t>(SEGMENT_ROWS, K - k0);
                if (!arrange_wide(&mask[(size_t)k0], rows, seg_slots)) {
                    fits = false;
                    return;
                }
                for (int q = 0; q < seg_slots.steps * 16; ++q) {
                    uint32_t before = 0;
                    for (int s = 4 * q; s < 4 * q + 4; ++s)
                        if (seg_slots.slot[s] >= 0) {
                            places[(size_t)(t * K + k0 + seg_slots.slot[s])] = {first * STEP_K + s, before};
                            before |= mask[(size_t)(k0 + seg_slots.slot[s])];
                        }
                }
                steps[(size_t)(t * nseg + seg)] = seg_slots.steps;
                first += seg_slots.steps;
            }
        }
    });
    if (!fits) return false;
    out.nsteps = 0;
    out.max_steps_per_tile = out.max_steps_per_segment = 0;
    std::vector<int64_t> first((size_t)nt + 1, 0);
    for (int64_t t = 0; t < nt; ++t) {
        int all = 0;
        for (int seg = 0; seg < nseg; ++seg) {
            all += steps[(size_t)(t * nseg + seg)];
            out.max_steps_per_segment = std::max(out.max_steps_per_segment, steps[(size_t)(t * nseg + seg)]);
        }
        out.max_steps_per_tile = std::max(out.max_steps_per_tile, all);
        first[(size_t)t + 1] = first[(size_t)t] + all;
    }
    out.nsteps = first[(size_t)nt];
    const bool strided = nt * out.max_steps_per_tile <= out.nsteps + out.nsteps / 2;
    out.tile_steps = strided ? out.max_steps_per_tile : 0;
    const int64_t records = std::max<int64_t>(1, strided ? nt * out.tile_steps : out.nsteps), at = wide_records_offset(nt, nseg);
    out.size = at + records * WIDE_RECORD_BYTES;
    out.bytes.reset(new uint8_t[(size_t)out.size]);
    std::memset(out.bytes.get(), 0, (size_t)at);
    int32_t* const rowsum = (int32_t*)out.bytes.get();
    int32_t* const bounds = (int32_t*)(out.bytes.get() + wide_bounds_offset(nt));
    uint8_t* const rec = out.bytes.get() + at;
    if (out.nsteps == 0) std::memset(rec, 0, (size_t)(records * WIDE_RECORD_BYTES));
    parallel_for(nt, grain, [&](int64_t begin, int64_t end) {
        for (int64_t t = begin; t < end; ++t) {
            const int64_t base = out.tile_steps ? t * out.tile_steps : first[(size_t)t];
            const int64_t count = first[(size_t)t + 1] - first[(size_t)t], room = out.tile_steps ? out.tile_steps : count;
            uint8_t* const mine = rec + base * WIDE_RECORD_BYTES;
            std::memset(mine, 0, (size_t)(room * WIDE_RECORD_BYTES));
            bounds[t * (nseg + 1)] = (int32_t)base;
            for (int seg = 0; seg < nseg; ++seg) bounds[t * (nseg + 1) + seg + 1] = bounds[t * (nseg + 1) + seg] + steps[(size_t)(t * nseg + seg)];
            // rows of padding slots: the residue that the octet lacks (see above)
            for (int seg = 0, s = 0; seg < nseg; ++seg) {
                const int rows = (int)std::min<int64_t>(SEGMENT_ROWS, K - (int64_t)seg * SEGMENT_ROWS);
                for (int i = 0; i < steps[(size_t)(t * nseg + seg)]; ++i, ++s) {
                    uint8_t* const r = mine + (int64_t)s * WIDE_RECORD_BYTES;
                    for (int z = 0; z < STEP_K; ++z) {
                        const int row = ((z & 7) + (z >> 3)) & 7;
                        set_row(r, z, row < rows ? row : 0);
                    }
                }
            }
            int32_t* const sum = rowsum + t * WIDE_ROWS;
            auto add = [&](const int64_t k, const int u, const int row, const int rows, const uint32_t v) {
                const Place& p = places[(size_t)(t * K + k)];
                const int z = p.slot & (STEP_K - 1), h = z >> 4 & 1, which = 8 * (z >> 5) + 2 * (z >> 2 & 3) + (int)(p.before >> u & 1);
                uint8_t* const r = mine + (int64_t)(p.slot / STEP_K) * WIDE_RECORD_BYTES;
                uint8_t* const val = r + (32 * h + row) * 16 + which;
                uint32_t* const sel = (uint32_t*)(r + WIDE_VAL_BYTES) + 2 * (32 * h + row);
                for (int i = 0; i < rows; ++i) {
                    val[16 * i] = (uint8_t)(v >> (8 * i));
                    sel[2 * i] |= (uint32_t)(z & 3) << (2 * which);
                    sum[row + i] += (int8_t)(v >> (8 * i));
                }
                set_row(r, z, (int)(k & (SEGMENT_ROWS - 1)));
            };
            for (int u = 0; u < units && t * units + u < b.block_rows; ++u) {
                const int64_t br = t * units + u;
                for (int64_t e = b.row_ptr[(size_t)br]; e < b.row_ptr[(size_t)br + 1]; ++e) {
                    uint32_t v;
                    std::memcpy(&v, &b.vals[(size_t)e * 4], 4);
                    const int64_t k = b.index[(size_t)e];
                    if (n4) {
                        add(k, u, 4 * u, 4, v);
                    } else {
                        for (int j = 0; j < 4; ++j)
                            if (v >> (8 * j) & 0xff) add(4 * k + j, u, u, 1, v >> (8 * j) & 0xff);
                    }
                }
            }
        }
    });
    return true;
}

}  // namespace spmm
