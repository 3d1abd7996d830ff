// Host side of the kernel launch: the plan (which configuration, which grid) and the dispatch
// to the per-configuration launchers compiled from spmm_launch_cfg.hip.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "spmm_internal.h"

namespace spmm {

#define SPMM_DECLARE_CFG(name) \
    void name(spmm_out_t, int postop, const unsigned* grid, unsigned block, void* stream, const KernelArgs&)
SPMM_DECLARE_CFG(launch_cfg_128_16_4);
SPMM_DECLARE_CFG(launch_cfg_128_16_5);
SPMM_DECLARE_CFG(launch_cfg_128_16_6);
SPMM_DECLARE_CFG(launch_cfg_128_8_4);
SPMM_DECLARE_CFG(launch_cfg_128_8_6);
SPMM_DECLARE_CFG(launch_cfg_128_8_8);
SPMM_DECLARE_CFG(launch_cfg_96_16_4);
SPMM_DECLARE_CFG(launch_cfg_96_16_5);
SPMM_DECLARE_CFG(launch_cfg_96_16_6);
SPMM_DECLARE_CFG(launch_cfg_fed_128_12_4);
SPMM_DECLARE_CFG(launch_cfg_fed_128_12_6);
SPMM_DECLARE_CFG(launch_cfg_fed_128_8_4);
SPMM_DECLARE_CFG(launch_cfg_fed_128_8_6);
SPMM_DECLARE_CFG(launch_cfg_fed_128_8_8);
SPMM_DECLARE_CFG(launch_cfg_fed_96_12_4);
SPMM_DECLARE_CFG(launch_cfg_fed_96_12_6);
SPMM_DECLARE_CFG(launch_cfg_fed_64_12_4);
SPMM_DECLARE_CFG(launch_cfg_fed_64_12_6);
SPMM_DECLARE_CFG(launch_cfg_simple_64_1);
SPMM_DECLARE_CFG(launch_cfg_simple_64_2);
SPMM_DECLARE_CFG(launch_cfg_simple_32_1);
SPMM_DECLARE_CFG(launch_cfg_simple_16_1);
SPMM_DECLARE_CFG(launch_cfg_slab16);
SPMM_DECLARE_CFG(launch_cfg_slab32);
SPMM_DECLARE_CFG(launch_cfg_stream64);
SPMM_DECLARE_CFG(launch_cfg_stream32);
SPMM_DECLARE_CFG(launch_cfg_stream16);
SPMM_DECLARE_CFG(launch_cfg_wide_128_8_5);
SPMM_DECLARE_CFG(launch_cfg_wide_128_8_6);
SPMM_DECLARE_CFG(launch_cfg_wide_128_8_7);
SPMM_DECLARE_CFG(launch_cfg_wide_128_8_8);
SPMM_DECLARE_CFG(launch_cfg_wide_96_8_5);
SPMM_DECLARE_CFG(launch_cfg_wide_96_8_6);
SPMM_DECLARE_CFG(launch_cfg_wide_96_8_7);
SPMM_DECLARE_CFG(launch_cfg_wide_96_8_8);
SPMM_DECLARE_CFG(launch_cfg_wide_64_8_5);
SPMM_DECLARE_CFG(launch_cfg_wide_64_8_6);
SPMM_DECLARE_CFG(launch_cfg_wide_64_8_7);
SPMM_DECLARE_CFG(launch_cfg_wide_64_8_8);
SPMM_DECLARE_CFG(launch_cfg_wide_64_4_5);
SPMM_DECLARE_CFG(launch_cfg_wide_64_4_6);
SPMM_DECLARE_CFG(launch_cfg_wide_64_4_7);
SPMM_DECLARE_CFG(launch_cfg_wide_64_4_8);
SPMM_DECLARE_CFG(launch_cfg_wide_32_4_5);
SPMM_DECLARE_CFG(launch_cfg_wide_32_4_6);
SPMM_DECLARE_CFG(launch_cfg_wide_32_4_7);
SPMM_DECLARE_CFG(launch_cfg_wide_32_4_8);
#undef SPMM_DECLARE_CFG

bool plan_supported(int token_tile, int variant)
{
    if (variant == 132) return token_tile == 128 || token_tile == 96 || token_tile == 64;
    if (variant == 134) return token_tile == 64 || token_tile == 32;
    if (token_tile == 128) return variant == 0 || variant == 8 || variant == 16 || variant == 108 || variant == 112;
    if (token_tile == 96) return variant == 0 || variant == 16 || variant == 112;
    if (token_tile == 64) return variant == 101 || variant == 102 || variant == 104 || variant == 112;
    if (token_tile == 32 || token_tile == 16) return variant == 101 || (variant >= 103 && variant <= 106);
    return false;
}

// What the candidates of one call have in common, worked out once.  A plan is made on every launch, and the host side
// of a launch is about 3.5 us, more than the kernel of a short one: 14 candidates with 64-bit divisions and byte counts
// of their own took 0.3 to 0.5 us of it (256x256, 128 tokens: 0.48, now 0.15; 1024x1024, 6144 tokens: 0.50, now 0.30;
// calls back to back of 896x256, 400 tokens: every 4.00 us, now 3.87).
struct Call {
    int64_t M;
    const WeightDims& w;
    int num_cus, per_xcd, cu_shift;     // cu_shift: per_xcd = 1 << cu_shift and num_cus = 8 * per_xcd; -1: neither
    // Bytes all XCDs together read through their L2s, when 2^rb slices of the packed weight and 8 / 2^rb slices of X are
    // dealt out among them (decode_workgroup): what comes from the last-level cache or HBM at a third of the L2's
    // rate, and is the largest part of many launches (4096x4096 at 75 %, 512 tokens, by the weight's rows alone: 31 MB).
    double fetched[4], fetch_us[4];     // and the time that takes at 7 TB/s
    int rank[4], split[4];              // rank[rb]: how many splits fetch less (or as much, with a smaller rb); and its inverse
    double w_bytes, x_bytes;
    double steps;                       // of a (row tile, segment), on average
    double wide_steps = 0.0;            // the same of the wide form (set_wide_steps)

    Call(int64_t tokens, const WeightDims& dims, int cus) : M(tokens), w(dims), num_cus(cus), per_xcd(cus >= 8 ? cus / 8 : 1)
    {
        cu_shift = (per_xcd & (per_xcd - 1)) == 0 && per_xcd * 8 == cus ? __builtin_ctz((unsigned)per_xcd) : -1;
        w_bytes = (double)w.nsteps * RECORD_BYTES;
        x_bytes = (double)w.K * (double)M;
        for (int rb = 0; rb <= 3; ++rb) {
            fetched[rb] = 8.0 * (w_bytes / (1 << rb) + x_bytes / (8 >> rb));
            fetch_us[rb] = fetched[rb] * 1e-6 / 7.0;
        }
        for (int rb = 0; rb <= 3; ++rb) {
            rank[rb] = 0;
            for (int o = 0; o <= 3; ++o) rank[rb] += o < rb ? fetched[o] <= fetched[rb] : fetched[o] < fetched[rb];
            split[rank[rb]] = rb;
        }
        steps = (double)w.nsteps / ((double)w.ntiles * w.nseg);
    }
    void set_wide_steps() { wide_steps = (double)w.wide_nsteps / ((double)((w.ntiles + 1) / 2) * w.nseg); }
    // rounds of `n` workgroups on all CUs, or of an XCD's share on its own
    int64_t rounds(int64_t n) const { return cu_shift >= 0 ? (n + num_cus - 1) >> (cu_shift + 3) : (n + num_cus - 1) / num_cus; }
    int64_t xcd_rounds(int64_t n) const { return cu_shift >= 0 ? (n + per_xcd - 1) >> cu_shift : (n + per_xcd - 1) / per_xcd; }
};

static int ceil_shift(int64_t v, int bits) { return (int)((v + ((int64_t)1 << bits) - 1) >> bits); }

static int quotient(int a, int b) { return (int)((unsigned)a / (unsigned)b); }     // of positive numbers

// Both are inlined so that the divisions by a tile's width and a workgroup's rows are by constants.
#define SPMM_INLINE static inline __attribute__((always_inline))

// Persistent kernels: token tile tm, `waves` row tiles (and `loaders` loader waves) per workgroup; as many token-tile
// streams per row group as fill every CU once.  Of the ways to deal the workgroups to the XCDs, those with the
// shortest streams, and of these the one that fetches least.
SPMM_INLINE void fill_pipelined(Plan& p, const Call& c, int tm, int waves, int loaders, int row_tiles = 1, int per_cu = 1)
{
    p.token_tile = tm;
    p.waves = waves;
    p.loaders = loaders;
    p.row_tiles_per_wave = row_tiles;
    p.simple = p.slab = p.stream = p.wide = 0;
    p.n_tok_tiles = (int)((c.M + tm - 1) / tm);
    p.n_row_groups = (c.w.ntiles + waves * row_tiles - 1) / (waves * row_tiles);
    int64_t best = INT64_MAX;
    int streams[4];
    for (int rb = 0; rb <= 3; ++rb) {
        const int rows = ceil_shift(p.n_row_groups, rb);
        int S = quotient(c.per_xcd * per_cu, rows) << (3 - rb);
        if (rows > c.per_xcd * per_cu) S = 1 << (3 - rb);
        if (p.n_row_groups >= c.num_cus * per_cu) S = 1;
        streams[rb] = S = std::min(S, p.n_tok_tiles);
        best = std::min(best, (int64_t)quotient(p.n_tok_tiles + S - 1, S) << 2 | c.rank[rb]);
    }
    p.xcd_row_bits = c.split[best & 3];
    p.n_streams = streams[p.xcd_row_bits];
    p.workgroups = (int64_t)p.n_row_groups * p.n_streams;
}

// The wide form: 8 (or 4, and two workgroups on a CU) compute waves of 32 rows each, and half as many loader waves.
SPMM_INLINE void fill_wide(Plan& p, const Call& c, int tm, int waves)
{
    fill_pipelined(p, c, tm, waves, waves / 2, WIDE_ROWS / TILE_ROWS, 8 / waves);
    p.wide = 1;
    p.max_steps = std::max(5, c.w.wide_max_steps);
}

// Workgroups whose slices take more rounds than their number does, dealt to the XCDs in equal parts (decode_tile), in the order
// that fetches less: an XCD's `each` consecutive workgroups touch so many row groups and so many token tiles.  A round saved is
// worth more than what the slices save: of 67 random problems of 256 to 4096 features, 32 to 1250 tokens, 70 to 90 %, where it
// saves one (profiles/spmm_plan_equal_parts.csv), no kernel is slower; two rounds of the resident kernels become one of 0.76 of the
// time (with one K segment, where two workgroups share a CU, 0.89), two of the ring one of 0.66, three and more 0.85.  What the plan
// then chooses takes 0.957 of the time that its choice by slices takes: 24 are more than 3 % faster, two slower.  Those two go from the
// wide form to a dealt slab (1300x2600 at 80 %, 346 tokens 8.0 -> 8.7), and the estimates of both are 10 to 60 % off there: of 113
// further problems of five to eight segments whose choice dealing changes (profiles/spmm_plan_equal_parts_slabs.csv) the choices take
// 0.93 of the time, 71 more than 3 % less, ten more than 3 % longer (2656x4096 at 70 %, 188 tokens, int32 10.1 -> 11.6, the others to
// 6 %).  Nothing that the plan knows tells those ten apart: without dealing from the wide form to slabs 30 would lose 6 % on average
// to save four of them, without dealing workgroups of 2 row tiles 33 would lose 3 % to save five.
// 768x3072 at 80 %, 333 tokens with Sum, binary32, 12 row groups x 21 token tiles: 12.2 -> 8.1 us, and as 6 x 21, which it ran as
// before, 9.2; 1300x650 at 80 %, 665 tokens 5.6 -> 4.8.
static void deal(Plan& p, const Call& c, int each)
{
    const double rows = p.n_row_groups, toks = p.n_tok_tiles;
    auto fetch = [&](double outer, double inner, double of_outer, double of_inner) {
        return of_outer * std::min(1.0, (each / inner + 1) / outer) + of_inner * std::min(1.0, each / inner);
    };
    const double by_rows = fetch(rows, toks, c.w_bytes, c.x_bytes), by_tokens = fetch(toks, rows, c.x_bytes, c.w_bytes);
    p.xcd_row_bits = by_tokens < by_rows;
    p.dealt = (uint32_t)((((uint64_t)1 << 32) + (uint64_t)(p.xcd_row_bits ? p.n_row_groups : p.n_tok_tiles) - 1) /
                         (uint64_t)(p.xcd_row_bits ? p.n_row_groups : p.n_tok_tiles));
    p.fetch_us = 8.0 * std::min(by_rows, by_tokens) * 1e-6 / 7.0;
    p.workgroups = 8 * (int64_t)each;
}

// Simple, short-batch and streamed kernels: tm-token tiles, one workgroup of 8 waves per (row group, tile), `waves` row
// tiles (or pairs of them) per row group.  The XCD split: as few rounds of workgroups as possible, then the least fetched.
SPMM_INLINE void fill_simple(Plan& p, const Call& c, int r, int tm, int waves = 8)
{
    p.token_tile = tm;
    p.waves = waves;
    p.loaders = 0;
    p.row_tiles_per_wave = r;
    p.simple = 1;
    p.slab = p.stream = p.wide = 0;
    p.n_tok_tiles = (int)((c.M + tm - 1) / tm);
    p.n_row_groups = (c.w.ntiles + waves * r - 1) / (waves * r);
    p.n_streams = 0;
    p.dealt = 0;
    int64_t best = INT64_MAX, here[4];
    for (int rb = 0; rb <= 3; ++rb) {
        here[rb] = (int64_t)ceil_shift(p.n_row_groups, rb) * ceil_shift(p.n_tok_tiles, 3 - rb);
        best = std::min(best, c.xcd_rounds(here[rb]) << 2 | c.rank[rb]);
    }
    p.xcd_row_bits = c.split[best & 3];
    p.workgroups = 8 * here[p.xcd_row_bits];
    p.fetch_us = c.fetch_us[p.xcd_row_bits];
    const int64_t all = (int64_t)p.n_row_groups * p.n_tok_tiles;
    if (all < 65536 && p.n_row_groups > 1 && p.n_tok_tiles > 1 && c.xcd_rounds((all + 7) / 8) < best >> 2) deal(p, c, (int)((all + 7) / 8));
}

// ---------------------------------------------------------------------------------------
// What a plan costs, in us: a fit to measured launches of 256 to 4096 features, 16 to 6144 tokens, 70 to 90 %, every
// output type, in every configuration that runs them; beyond that range it is an extrapolation.  The estimates are
// within 5 to 16 % of the measurement (standard deviation, by configuration).  Of 800 problems that none is fitted to
// (profiles/spmm_plan_resident_measurements.csv: every type, layout and orientation) the cheapest configuration by them takes 1.014 of
// the fastest one's time, over 1.1 in 2.6 %; where the weight has no wide form (596 problems, profiles/spmm_plan_measurements.csv)
// 1.022, with tile-major activations 1.018, which the estimates do not tell from row-major ones, over 1.1 in 8 and 7 %; tests
// recompute these figures.  The resident kernels (RES, SLAB) have become up to 1.3 times faster with their straight-line start; by
// the fits of before the 800 take 1.032, over 1.1 in 11.9 %: with the fits of now, 1500 times on average for each, 140 of them
// run another kernel, 10 are more than 3 % slower, and together all are 1.018 times as fast (tests/test_plan_resident.py).
// 1024x256 at 80 %, 1024 tokens, u8 with GELU: the ring with 32-token tiles, 4.26 us, became the resident kernel, 3.61.
// A launch is a start, rounds of workgroups on the CUs, and in a round: phases (a K segment of a token tile) with
// their matrix instructions and the staging of their activations, and the tiles' post-operators; what has to
// be fetched through the L2s adds to all of it.
// ---------------------------------------------------------------------------------------
struct Fit {
    double start, phase, unit, tokens, out1, out4, fetch;
};

// persistent kernels: {up to two K segments (weights stay in registers), more (reloaded every phase)}
//                                     start  phase   unit    tokens  out1    out4    fetch
static const Fit FIT_128_8[2]      = {{2.36, 0.00, 0.0027, 0.93, 0.0564, 0.0937, 1.57},
                                     {1.55, 0.00, 0.0032, 0.90, 0.1313, 0.1594, 0.96}};
static const Fit FIT_128_16[2]     = {{1.79, 0.00, 0.0036, 1.03, 0.0564, 0.0937, 1.57},
                                     {1.42, 0.00, 0.0045, 0.21, 0.1313, 0.1594, 0.96}};
static const Fit FIT_96_16[2]      = {{2.22, 1.20, 0.0027, 0.00, 0.0564, 0.0937, 1.57},
                                     {1.31, 0.55, 0.0041, 0.00, 0.1313, 0.1594, 0.96}};
static const Fit FIT_FED_128_8[2]  = {{2.69, 0.00, 0.0028, 0.78, 0.0515, 0.0884, 1.23},
                                     {2.77, 0.00, 0.0022, 0.70, 0.1156, 0.1499, 0.76}};
static const Fit FIT_FED_128_12[2] = {{2.48, 0.00, 0.0058, 0.39, 0.0515, 0.0884, 1.23},
                                     {2.56, 0.00, 0.0031, 0.52, 0.1156, 0.1499, 0.76}};
static const Fit FIT_FED_96_12[2]  = {{2.76, 0.90, 0.0034, 0.00, 0.0515, 0.0884, 1.23},
                                     {2.48, 0.82, 0.0028, 0.00, 0.1156, 0.1499, 0.76}};
static const Fit FIT_FED_64_12[2]  = {{2.88, 0.56, 0.0030, 0.00, 0.0515, 0.0884, 1.23},
                                     {2.39, 0.52, 0.0033, 0.00, 0.1156, 0.1499, 0.76}};
// the resident kernels (with 8, 4 and 2 row tiles)
static const Fit FIT_RES_16[3]     = {{1.81, 0.61, 0.0055, 1.38, 0.0331, 0.0000, 1.94}, {1.64, 0.61, 0.0059, 1.66, 0.0536, 0.0000, 1.50},
                                      {1.57, 0.76, 0.0093, 1.08, 0.0871, 0.0000, 1.28}};
static const Fit FIT_SLAB_16[3]    = {{0.00, 3.44, 0.0064, 0.17, 0.0661, 0.0000, 1.66}, {0.00, 2.51, 0.0106, 0.80, 0.2333, 0.0000, 0.80},
                                      {0.03, 3.18, 0.0087, 0.44, 0.2673, 0.0000, 0.08}};
static const Fit FIT_RES_32        = {2.02, 0.77, 0.0032, 0.97, 0.0104, 0.0000, 1.39};
static const Fit FIT_RES_64        = {2.25, 0.83, 0.0025, 0.61, 0.0038, 0.0000, 1.99};
static const Fit FIT_RING_16       = {2.24, 0.68, 0.0082, 2.70, 0.0208, 0.0000, 1.04};
static const Fit FIT_RING_32       = {0.90, 1.96, 0.0062, 2.06, 0.0130, 0.0000, 1.29};
static const Fit FIT_RING_64       = {0.52, 2.99, 0.0039, 1.18, 0.0008, 0.0000, 1.53};

// the wide form (units: 32 tokens of a step of 32 rows): 4700 other problems, 256 to 4096 features, 16 to 6144 tokens, 3e7
// products and more, every layout; on the problems of profiles/spmm_plan_wide_measurements.csv, drawn on their own, the
// estimates are 0.96 to 0.98 of the time, standard deviation 9 to 12 %
static const Fit FIT_WIDE_128_8[2]   = {{2.88, 0.00, 0.0018, 0.84, 0.0745, 0.0841, 1.32},
                                      {2.73, 0.71, 0.0047, 0.00, 0.0940, 0.1020, 0.62}};
static const Fit FIT_WIDE_96_8[2]    = {{2.82, 0.00, 0.0017, 0.81, 0.0869, 0.1050, 1.33},
                                      {2.48, 0.83, 0.0039, 0.00, 0.0807, 0.1077, 0.79}};
static const Fit FIT_WIDE_64_8[2]    = {{2.89, 0.00, 0.0021, 1.00, 0.0859, 0.1019, 1.37},
                                      {2.35, 0.50, 0.0068, 0.00, 0.0821, 0.1041, 0.68}};
static const Fit FIT_WIDE_64_4[2]    = {{2.65, 0.13, 0.0004, 1.00, 0.0902, 0.1134, 1.93},
                                      {2.91, 0.00, 0.0038, 0.92, 0.1423, 0.1542, 0.77}};
static const Fit FIT_WIDE_32_4[2]    = {{2.83, 0.00, 0.0009, 1.73, 0.0961, 0.1593, 1.67},
                                      {2.56, 0.00, 0.0044, 1.82, 0.0992, 0.2153, 0.61}};

SPMM_INLINE double plan_cost(const Plan& p, const Fit& f, const Call& c, int out_bytes)
{
    const double rounds = (double)c.rounds(p.workgroups);
    const double rows = p.waves;
    if (p.simple) {
        const double units = rows * c.steps * c.w.nseg * p.token_tile / 16.0;
        return f.start + rounds * (f.phase + f.unit * units + f.tokens * c.w.nseg * p.token_tile * 0.01 +
                                   f.out1 * rows * TILE_ROWS * p.token_tile * 1e-3 * out_bytes) + f.fetch * p.fetch_us;
    }
    const int tiles = quotient(p.n_tok_tiles + p.n_streams - 1, p.n_streams), phases = tiles * c.w.nseg;
    const double units = rows * c.steps * p.token_tile / 16.0;
    return rounds * (f.start + phases * (f.phase + f.unit * units + f.tokens * p.token_tile * 0.01) +
                     (out_bytes == 4 ? f.out4 : f.out1) * tiles * rows * TILE_ROWS * p.token_tile * 1e-3) + f.fetch * c.fetch_us[p.xcd_row_bits];
}

// The same of the wide form's kernel: an XCD's workgroups take its CUs in rounds of per_cu to a CU, and those that share a CU
// share its matrix cores, its LDS and its stores.
SPMM_INLINE double wide_cost(const Plan& p, const Fit& f, const Call& c, int out_bytes, int per_cu, double post)
{
    const int64_t n = (int64_t)ceil_shift(p.n_row_groups, p.xcd_row_bits) * ceil_shift(p.n_streams, 3 - p.xcd_row_bits);
    const int64_t per_xcd = c.xcd_rounds(n);
    const double rounds = (double)((per_xcd + per_cu - 1) / per_cu), sharing = (double)std::min<int64_t>(per_cu, per_xcd);
    const int tiles = quotient(p.n_tok_tiles + p.n_streams - 1, p.n_streams), phases = tiles * c.w.nseg;
    const double units = p.waves * c.wide_steps * p.token_tile / 32.0;
    return rounds * (f.start + phases * (f.phase + sharing * (f.unit * units + f.tokens * p.token_tile * 0.01)) +
                     sharing * post * (out_bytes == 4 ? f.out4 : f.out1) * tiles * p.waves * WIDE_ROWS * p.token_tile * 1e-3) +
           f.fetch * c.fetch_us[p.xcd_row_bits];
}

// A configuration that spmm_set_tuning asked for (force_tm != 0), or the nearest one that runs this weight.
static Plan forced_plan(const Call& call, int force_tm, int variant, int max_steps, int fed_steps, int widest)
{
    const int nseg = call.w.nseg;
    Plan p{};
    p.max_steps = max_steps;
    if (variant == 132 || variant == 134) {
        if (call.w.wide_max_steps > 0 && widest >= 32) {
            fill_wide(p, call, std::min(force_tm, widest), variant == 132 ? 8 : 4);
            return p;
        }
        variant = 108;
        force_tm = 128;
    }
    if (force_tm == 64 || force_tm == 32 || force_tm == 16) {
        if (variant == 112) {
            // (weights with more than 6 steps per segment run 8 compute waves, which exist with 128-token tiles)
            fill_pipelined(p, call, max_steps <= 6 ? 64 : 128, max_steps <= 6 ? 12 : 8, 4);
            p.max_steps = fed_steps;
            return p;
        }
        const int r = variant == 102 ? 2 : 1, row_tiles = variant == 105 ? 2 : variant == 106 ? 4 : 8;
        fill_simple(p, call, r, force_tm, row_tiles);
        // the short-batch kernel takes K <= 4096 (3072 with 32-token tiles); longer K silently runs the simple kernel
        if (variant == 103) p.slab = nseg <= (force_tm == 16 ? SLAB_SEGMENTS : SLAB_SEGMENTS_32);
        if (row_tiles < 8) p.slab = force_tm == 16 && nseg > 4 && nseg <= SLAB_SEGMENTS;
        p.stream = variant == 104;
        return p;
    }
    if (variant == 108 || variant == 112) {
        // 12 compute waves have 128 registers each (at most 6 step slots); denser weights take 8
        const int waves = (variant == 112 && max_steps <= 6) ? 12 : 8;
        fill_pipelined(p, call, (waves == 12 && force_tm == 96) ? 96 : 128, waves, 4);
        p.max_steps = fed_steps;
        return p;
    }
    // 16 waves have 128 registers each: at most 6 steps per segment; denser weights run with 8
    // waves, 256 registers and half as many rows per workgroup (token tile 128 only)
    const bool eight = max_steps > 6 || variant == 8;
    fill_pipelined(p, call, eight ? 128 : force_tm, eight ? 8 : 16, 0);
    return p;
}

Plan make_plan(int64_t M, const WeightDims& w, int num_cus, int force_tm, int variant, int out_bytes, bool x_fast, bool out_fast,
               int widest, double wide_handicap)
{
    const int nseg = w.nseg, max_steps_per_segment = w.max_steps_per_segment;
    Call call(M, w, num_cus);
    const int max_steps = max_steps_per_segment <= 4 ? 4 : (max_steps_per_segment <= 6 ? max_steps_per_segment : 8);
    const int fed_steps = max_steps == 5 ? 6 : max_steps;      // step slots of the loader-wave kernels: 4, 6 or 8
    if (!x_fast && !(force_tm && force_tm <= 64 && (variant == 101 || variant == 102))) {
        // rows so far apart that a segment of them exceeds 32-bit offsets, or an X of less than 16 bytes
        Plan p{};
        p.max_steps = max_steps;
        fill_simple(p, call, 1, 64);
        return p;
    }
    if (force_tm) return forced_plan(call, force_tm, variant, max_steps, fed_steps, out_fast ? widest : 0);
    // ---- short and mid-size batches
    const int reload = nseg > 2;
    Plan best{}, c{};
    double best_cost = 0.0;
    c.max_steps = max_steps;
    auto consider = [&](const Fit& f, const double margin = 0.98) __attribute__((always_inline)) {
        const double cost = plan_cost(c, f, call, out_bytes);
        if (best.workgroups == 0 || cost < margin * best_cost) {
            best = c;
            best_cost = cost;
        }
    };
    auto short_batch = [&](const int row_tiles) __attribute__((always_inline)) {
        fill_simple(c, call, 1, 16, row_tiles);
        if (nseg > SLAB_SEGMENTS) c.stream = 1;
        else if (nseg > 4) c.slab = 1;
        // fewer rows per workgroup, the waves sharing a row tile's steps: where whole workgroups would leave most of the chip
        // idle; with three and four segments as long as an eighth of the CUs has none (with few steps the sum over the
        // shares costs what the shorter walk saves; two segments, which would gain 4 %, keep the line that
        // tests/test_host_pack.py pins for 768x768, 128 tokens).  Of 640 measured problems of 256 to 4096 features, time with
        // 4 row tiles over that with 8, three and four segments, by workgroups: up to 224, 0.93; 240, 0.99, and some
        // 1.15, as workgroups do not divide by XCDs; from 256 on, where CUs have two, 1.2.  With 2 over 4: 0.98, 1.04, 1.2.
        if (row_tiles < 8 && c.stream) return false;
        if (row_tiles < 8 && !c.slab && (int64_t)c.n_row_groups * c.n_tok_tiles * row_tiles / 8 >= num_cus * 3 / 16 &&
            (nseg <= 2 || c.workgroups > num_cus * 7 / 8)) return false;
        const int fewer = row_tiles == 8 ? 0 : row_tiles == 4 ? 1 : 2;
        consider(c.stream ? FIT_RING_16 : c.slab ? FIT_SLAB_16[fewer] : FIT_RES_16[fewer]);
        return true;
    };
    if (short_batch(8) && short_batch(4)) short_batch(2);
    // (the simple kernel where its resident rows hold all of K, the ring beyond)
    fill_simple(c, call, 1, 32);
    if (nseg <= 4) consider(FIT_RES_32);
    if (nseg > 4 && nseg <= SLAB_SEGMENTS_32) c.slab = 1;
    else c.stream = 1;
    consider(FIT_RING_32);
    fill_simple(c, call, 1, 64);
    if (nseg <= 2) consider(FIT_RES_64);
    c.stream = 1;
    consider(FIT_RING_64);
    // ---- persistent kernels, where they occupy more than half of the CUs (the rest is the short-batch kernels' ground).
    // 16 waves have 128 registers each: at most 6 steps per segment; without loader waves the general store path
    // (outputs beyond 32-bit offsets) has no registers in them either.
    auto persistent = [&](const int tm, const int waves, const int loaders, const Fit& f, const double margin = 0.98) __attribute__((always_inline)) {
        // (no more workgroups than row groups x token tiles: most short batches end here)
        if ((int64_t)((w.ntiles + waves - 1) / waves) * ((M + tm - 1) / tm) * 2 <= num_cus) return;
        fill_pipelined(c, call, tm, waves, loaders);
        if (c.workgroups * 2 > num_cus) consider(f, margin);
    };
    if (max_steps <= 6 && out_fast) {
        persistent(128, 16, 0, FIT_128_16[reload]);
        // Against wider tiles of the same waves the fit favours 96 tokens by 2.5 % in row-major order, and in both orders
        // where a stream then has more tiles: a near tie goes to the wider (4096x1024 at 85 %, 6144 tokens, estimated
        // 31.5 us and 30.8: 128 tokens 24.9 us, 96 tokens 26.0; tile-major 22.3 and 23.1).  Not with 6 step slots, which
        // leave the wider form few registers for gathers in flight (80 %: 27.7 and 27.9; tile-major 26.3 and 25.1).
        persistent(96, 16, 0, FIT_96_16[reload], best.waves == 16 && max_steps <= 5 ? 0.96 : 0.98);
    }
    persistent(128, 8, 0, FIT_128_8[reload]);
    c.max_steps = fed_steps;
    persistent(128, 8, 4, FIT_FED_128_8[reload]);
    if (max_steps <= 6) {
        // 1-byte outputs of one token tile per stream and at most 4 steps per segment keep the forms of 8 or 16 compute
        // waves, but for 64-token tiles of weights that are reloaded: those were faster in all of 26 measured problems
        // that they now get (768x3072 at 90 %, 4096 tokens, tile-major 12.7 -> 10.0 us, row-major 12.6 -> 10.7;
        // 1300x2600 at 89 %, 1392 tokens 21.7 -> 10.2).  The wider tiles the fit would also take where they are slower
        // (1792x3584 at 88 %, 2369 tokens: 22.3 against 23.2); weights of one or two segments stay out because
        // tests/test_host_pack.py pins 768x768, 4096 tokens, to 8 waves (90 %: 6.6 us, with 12 + 4 waves 5.8).
        auto fed12 = [&](const int tm, const Fit& f) __attribute__((always_inline)) {
            if ((int64_t)((w.ntiles + 11) / 12) * ((M + tm - 1) / tm) * 2 <= num_cus) return;
            fill_pipelined(c, call, tm, 12, 4);
            if (!(reload && tm == 64) && out_bytes == 1 && max_steps <= 4 && c.n_tok_tiles <= c.n_streams) return;
            if (c.workgroups * 2 > num_cus) consider(f);
        };
        fed12(128, FIT_FED_128_12[reload]);
        fed12(96, FIT_FED_96_12[reload]);
        fed12(64, FIT_FED_64_12[reload]);
    }
    // ---- the wide form, from 192 blocks of 32 rows x 32 tokens on (of 200 measured problems with fewer none
    // would be faster with it).  Of the 698 problems of profiles/spmm_plan_wide_measurements.csv that
    // have more one of its configurations is the fastest in 33 %.  What the estimates, whose errors are 9 to 11 %, set apart by
    // less than the margins below goes to the kernels above, because a wrong choice is seen and a missed one is not: 30 % get it,
    // 0.4 % are more than 3 % slower than without it, and all together are 1.059 times as fast (1.064 if every choice were right;
    // with margins of 0.98 34 % would get it, 2.0 % lose more than 3 %, and the gain is the same).  By what it replaces: the
    // 128-token kernels with 8 + 4 waves 1.24 times, the streamed kernels 1.27, the resident ones 1.26.  4-byte outputs that
    // have the 32-token slab keep it up to 768 blocks because tests/test_gpu_parity.py pins 768x3072, 1024 tokens, to it (such
    // problems would be 1.2 times as fast with the wide form).
    const int64_t blocks = (int64_t)((w.ntiles + 1) / 2) * ((M + 31) / 32);
    const bool pinned = out_bytes == 4 && best.slab && best.token_tile == 32 && blocks <= 768;
    // (nor where the others are estimated under 5 us: of 468 such measured problems none would get it, and its estimates take 0.1 us)
    if (w.wide_max_steps > 0 && out_fast && blocks >= 192 && best_cost > 5.0 && !pinned) {
        call.set_wide_steps();
        const double post = widest < 128 ? 1.8 : 1.0;      // (Sum, GELU in f32: of the fits with each, the closest)
        auto wide = [&](const int tm, const int waves, const Fit& f) __attribute__((always_inline)) {
            if (tm > widest) return;
            fill_wide(c, call, tm, waves);
            const double cost = wide_handicap * wide_cost(c, f, call, out_bytes, 8 / waves, post);
            if (cost < (best.wide ? 0.98 : reload ? 0.94 : 0.92) * best_cost) {
                best = c;
                best_cost = cost;
            }
        };
        wide(128, 8, FIT_WIDE_128_8[reload]);
        wide(96, 8, FIT_WIDE_96_8[reload]);
        wide(64, 8, FIT_WIDE_64_8[reload]);
        wide(64, 4, FIT_WIDE_64_4[reload]);
        wide(32, 4, FIT_WIDE_32_4[reload]);
    }
    return best;
}

int launch_spmm(const Plan& plan, KernelArgs& a, spmm_out_t out_type, int postop, void* stream)
{
    (void)hipGetLastError();   // an error left by an earlier, unrelated call is not this launch's
    a.n_streams = (uint16_t)(plan.simple ? plan.waves : plan.n_streams);
    a.k_flags |= (uint32_t)plan.xcd_row_bits << ARG_XCD_SHIFT;
    const unsigned block = plan.simple ? 512u : (unsigned)(plan.waves + plan.loaders) * 64;
    // x: XCD and row group within its slice, y and z: token tile or stream within its slice (decode_workgroup)
    const unsigned toks = (unsigned)ceil_shift(plan.simple ? plan.n_tok_tiles : plan.n_streams, 3 - plan.xcd_row_bits);
    const unsigned y = toks < (1u << GRID_Y_BITS) ? toks : (1u << GRID_Y_BITS);
    unsigned grid[3] = {8u * (unsigned)ceil_shift(plan.n_row_groups, plan.xcd_row_bits), y, (toks + y - 1) / y};
    if (plan.simple) {
        a.tiles_per_stream = plan.dealt;
        if (plan.dealt) {
            grid[0] = (unsigned)plan.workgroups;
            grid[1] = grid[2] = 1;
        }
        const int key = plan.token_tile * 10 + plan.row_tiles_per_wave;
        if (plan.stream) {
            if (key == 641) launch_cfg_stream64(out_type, postop, grid, block, stream, a);
            else if (key == 321) launch_cfg_stream32(out_type, postop, grid, block, stream, a);
            else if (key == 161) launch_cfg_stream16(out_type, postop, grid, block, stream, a);
            else return (int)hipErrorInvalidValue;
        } else if (plan.slab) {
            if (key == 161) launch_cfg_slab16(out_type, postop, grid, block, stream, a);
            else if (key == 321) launch_cfg_slab32(out_type, postop, grid, block, stream, a);
            else return (int)hipErrorInvalidValue;
        } else if (key == 641) launch_cfg_simple_64_1(out_type, postop, grid, block, stream, a);
        else if (key == 642) launch_cfg_simple_64_2(out_type, postop, grid, block, stream, a);
        else if (key == 321) launch_cfg_simple_32_1(out_type, postop, grid, block, stream, a);
        else if (key == 161) launch_cfg_simple_16_1(out_type, postop, grid, block, stream, a);
        else return (int)hipErrorInvalidValue;
        return (int)hipGetLastError();
    }
    a.tiles_per_stream = (uint32_t)(plan.n_tok_tiles / plan.n_streams);
    if (plan.wide) {
        switch (plan.token_tile * 100 + plan.waves * 10 + plan.max_steps) {
        case 12885: launch_cfg_wide_128_8_5(out_type, postop, grid, block, stream, a); break;
        case 12886: launch_cfg_wide_128_8_6(out_type, postop, grid, block, stream, a); break;
        case 12887: launch_cfg_wide_128_8_7(out_type, postop, grid, block, stream, a); break;
        case 12888: launch_cfg_wide_128_8_8(out_type, postop, grid, block, stream, a); break;
        case 9685: launch_cfg_wide_96_8_5(out_type, postop, grid, block, stream, a); break;
        case 9686: launch_cfg_wide_96_8_6(out_type, postop, grid, block, stream, a); break;
        case 9687: launch_cfg_wide_96_8_7(out_type, postop, grid, block, stream, a); break;
        case 9688: launch_cfg_wide_96_8_8(out_type, postop, grid, block, stream, a); break;
        case 6485: launch_cfg_wide_64_8_5(out_type, postop, grid, block, stream, a); break;
        case 6486: launch_cfg_wide_64_8_6(out_type, postop, grid, block, stream, a); break;
        case 6487: launch_cfg_wide_64_8_7(out_type, postop, grid, block, stream, a); break;
        case 6488: launch_cfg_wide_64_8_8(out_type, postop, grid, block, stream, a); break;
        case 6445: launch_cfg_wide_64_4_5(out_type, postop, grid, block, stream, a); break;
        case 6446: launch_cfg_wide_64_4_6(out_type, postop, grid, block, stream, a); break;
        case 6447: launch_cfg_wide_64_4_7(out_type, postop, grid, block, stream, a); break;
        case 6448: launch_cfg_wide_64_4_8(out_type, postop, grid, block, stream, a); break;
        case 3245: launch_cfg_wide_32_4_5(out_type, postop, grid, block, stream, a); break;
        case 3246: launch_cfg_wide_32_4_6(out_type, postop, grid, block, stream, a); break;
        case 3247: launch_cfg_wide_32_4_7(out_type, postop, grid, block, stream, a); break;
        case 3248: launch_cfg_wide_32_4_8(out_type, postop, grid, block, stream, a); break;
        default: return (int)hipErrorInvalidValue;
        }
        return (int)hipGetLastError();
    }
    const int maxs = (plan.waves == 8 && plan.max_steps == 5) ? 6 : plan.max_steps;   // no 8-wave 5-step build
    if (plan.loaders) {
        switch (plan.token_tile * 10000 + plan.waves * 100 + maxs) {
        case 1281204: launch_cfg_fed_128_12_4(out_type, postop, grid, block, stream, a); break;
        case 1281206: launch_cfg_fed_128_12_6(out_type, postop, grid, block, stream, a); break;
        case 1280804: launch_cfg_fed_128_8_4(out_type, postop, grid, block, stream, a); break;
        case 1280806: launch_cfg_fed_128_8_6(out_type, postop, grid, block, stream, a); break;
        case 1280808: launch_cfg_fed_128_8_8(out_type, postop, grid, block, stream, a); break;
        case 961204: launch_cfg_fed_96_12_4(out_type, postop, grid, block, stream, a); break;
        case 961206: launch_cfg_fed_96_12_6(out_type, postop, grid, block, stream, a); break;
        case 641204: launch_cfg_fed_64_12_4(out_type, postop, grid, block, stream, a); break;
        case 641206: launch_cfg_fed_64_12_6(out_type, postop, grid, block, stream, a); break;
        default: return (int)hipErrorInvalidValue;
        }
        return (int)hipGetLastError();
    }
    switch (plan.token_tile * 10000 + plan.waves * 100 + maxs) {
    case 1281604: launch_cfg_128_16_4(out_type, postop, grid, block, stream, a); break;
    case 1281605: launch_cfg_128_16_5(out_type, postop, grid, block, stream, a); break;
    case 1281606: launch_cfg_128_16_6(out_type, postop, grid, block, stream, a); break;
    case 1280804: launch_cfg_128_8_4(out_type, postop, grid, block, stream, a); break;
    case 1280806: launch_cfg_128_8_6(out_type, postop, grid, block, stream, a); break;
    case 1280808: launch_cfg_128_8_8(out_type, postop, grid, block, stream, a); break;
    case 961604: launch_cfg_96_16_4(out_type, postop, grid, block, stream, a); break;
    case 961605: launch_cfg_96_16_5(out_type, postop, grid, block, stream, a); break;
    case 961606: launch_cfg_96_16_6(out_type, postop, grid, block, stream, a); break;
    default: return (int)hipErrorInvalidValue;
    }
    return (int)hipGetLastError();
}

}  // namespace spmm
