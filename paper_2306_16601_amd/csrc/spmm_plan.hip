// Host side of the kernel launch: the plan (which configuration, which grid) and the dispatch
// to the per-configuration launchers compiled from spmm_launch_cfg.hip.
#include <hip/hip_runtime.h>

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
#undef SPMM_DECLARE_CFG

bool plan_supported(int token_tile, int variant)
{
    if (token_tile == 128) return variant == 0 || variant == 8 || variant == 16 || variant == 108 || variant == 112;
    if (token_tile == 96) return variant == 0 || variant == 16 || variant == 112;
    if (token_tile == 64) return variant == 101 || variant == 102 || variant == 104 || variant == 112;
    if (token_tile == 32 || token_tile == 16) return variant == 101 || (variant >= 103 && variant <= 106);
    return false;
}

// Bytes all XCDs together read through their L2s, when 2^row_bits slices of the packed weight and 8 / 2^row_bits
// slices of X are dealt out among them (decode_workgroup): what comes from the last-level cache or HBM at a
// third of the L2's rate, and is the largest part of many launches (4096x4096 at 75 %, 512 tokens, by the weight's
// rows alone: 31 MB).
static double fetched_bytes(const WeightDims& w, int64_t M, int row_bits)
{
    const double w_bytes = (double)w.nsteps * RECORD_BYTES, x_bytes = (double)w.K * (double)M;
    return 8.0 * (w_bytes / (1 << row_bits) + x_bytes / (8 >> row_bits));
}

static int ceil_shift(int64_t v, int bits) { return (int)((v + ((int64_t)1 << bits) - 1) >> bits); }

// Persistent kernels: token tile tm, `waves` row tiles (and `loaders` loader waves) per workgroup; as many token-tile
// streams per row group as fill every CU once.  Of the ways to deal the workgroups to the XCDs, those with the
// shortest streams, and of these the one that fetches least.
static void fill_pipelined(Plan& p, int64_t M, const WeightDims& w, int num_cus, int tm, int waves, int loaders)
{
    p.token_tile = tm;
    p.waves = waves;
    p.loaders = loaders;
    p.row_tiles_per_wave = 1;
    p.simple = p.slab = p.stream = 0;
    p.n_tok_tiles = (int)((M + tm - 1) / tm);
    p.n_row_groups = (w.ntiles + waves - 1) / waves;
    const int per_xcd = num_cus >= 8 ? num_cus / 8 : 1;
    int best_tiles = 0;
    double best_bytes = 0.0;
    for (int rb = 0; rb <= 3; ++rb) {
        const int rows = ceil_shift(p.n_row_groups, rb);
        int S = (rows >= per_xcd ? 1 : per_xcd / rows) << (3 - rb);
        if (p.n_row_groups >= num_cus) S = 1;
        if (S > p.n_tok_tiles) S = p.n_tok_tiles;
        const int tiles = (p.n_tok_tiles + S - 1) / S;
        const double bytes = fetched_bytes(w, M, rb);
        if (rb == 0 || tiles < best_tiles || (tiles == best_tiles && bytes < best_bytes)) {
            best_tiles = tiles;
            best_bytes = bytes;
            p.n_streams = S;
            p.xcd_row_bits = rb;
        }
    }
    p.workgroups = (int64_t)p.n_row_groups * p.n_streams;
}

// Simple, short-batch and streamed kernels: tm-token tiles, one workgroup of 8 waves per (row group, tile), `waves` row
// tiles (or pairs of them) per row group.  The XCD split: as few rounds of workgroups as possible, then the least fetched.
static void fill_simple(Plan& p, int64_t M, const WeightDims& w, int num_cus, int r, int tm, int waves = 8)
{
    p.token_tile = tm;
    p.waves = waves;
    p.loaders = 0;
    p.row_tiles_per_wave = r;
    p.simple = 1;
    p.slab = p.stream = 0;
    p.n_tok_tiles = (int)((M + tm - 1) / tm);
    p.n_row_groups = (w.ntiles + waves * r - 1) / (waves * r);
    p.n_streams = 0;
    const int64_t per_xcd = num_cus >= 8 ? num_cus / 8 : 1;
    int64_t best_rounds = 0;
    double best_bytes = 0.0;
    for (int rb = 0; rb <= 3; ++rb) {
        const int64_t here = (int64_t)ceil_shift(p.n_row_groups, rb) * ceil_shift(p.n_tok_tiles, 3 - rb);
        const int64_t rounds = (here + per_xcd - 1) / per_xcd;
        const double bytes = fetched_bytes(w, M, rb);
        if (rb == 0 || rounds < best_rounds || (rounds == best_rounds && bytes < best_bytes)) {
            best_rounds = rounds;
            best_bytes = bytes;
            p.xcd_row_bits = rb;
            p.workgroups = 8 * here;
        }
    }
}

// ---------------------------------------------------------------------------------------
// What a plan costs, in us: a fit to measured launches (280 problems of 256 to 4096 features, 16 to 6144
// tokens, 70 to 90 %, every output type, in every configuration that runs them; the fit is within 10 to 15 %
// of the measurement, and the cheapest configuration by it within 3 to 4 % of the fastest one).
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
static const Fit FIT_RES_16        = {2.18, 1.27, 0.0107, 1.20, 0.0091, 0.0000, 1.18};
static const Fit FIT_RES_32        = {2.56, 1.07, 0.0049, 1.16, 0.0067, 0.0000, 1.37};
static const Fit FIT_RES_64        = {3.71, 0.00, 0.0039, 1.15, 0.0054, 0.0000, 1.70};
static const Fit FIT_SLAB_16       = {0.83, 2.22, 0.0133, 2.73, 0.0271, 0.0000, 0.00};
static const Fit FIT_RING_16       = {2.24, 0.68, 0.0082, 2.70, 0.0208, 0.0000, 1.04};
static const Fit FIT_RING_32       = {0.90, 1.96, 0.0062, 2.06, 0.0130, 0.0000, 1.29};
static const Fit FIT_RING_64       = {0.52, 2.99, 0.0039, 1.18, 0.0008, 0.0000, 1.53};

static double plan_cost(const Plan& p, const Fit& f, const WeightDims& w, int64_t M, int num_cus, int out_bytes)
{
    const double rounds = (double)((p.workgroups + num_cus - 1) / num_cus);
    const double fetch = fetched_bytes(w, M, p.xcd_row_bits) * 1e-6 / 7.0;          // us at 7 TB/s
    const double steps = (double)w.nsteps / ((double)w.ntiles * w.nseg);            // of a (row tile, segment)
    const double rows = p.waves;
    if (p.simple) {
        const double units = rows * steps * w.nseg * p.token_tile / 16.0;
        return f.start + rounds * (f.phase + f.unit * units + f.tokens * w.nseg * p.token_tile * 0.01 +
                                   f.out1 * rows * TILE_ROWS * p.token_tile * 1e-3 * out_bytes) + f.fetch * fetch;
    }
    const int tiles = (p.n_tok_tiles + p.n_streams - 1) / p.n_streams, phases = tiles * w.nseg;
    const double units = rows * steps * p.token_tile / 16.0;
    return rounds * (f.start + phases * (f.phase + f.unit * units + f.tokens * p.token_tile * 0.01) +
                     (out_bytes == 4 ? f.out4 : f.out1) * tiles * rows * TILE_ROWS * p.token_tile * 1e-3) + f.fetch * fetch;
}

Plan make_plan(int64_t M, const WeightDims& w, int num_cus, int force_tm, int variant, int out_bytes, bool x_fast, bool out_fast)
{
    const int nseg = w.nseg, max_steps_per_segment = w.max_steps_per_segment;
    Plan p{};
    const int max_steps = max_steps_per_segment <= 4 ? 4 : (max_steps_per_segment <= 6 ? max_steps_per_segment : 8);
    const int fed_steps = max_steps == 5 ? 6 : max_steps;      // step slots of the loader-wave kernels: 4, 6 or 8
    p.max_steps = max_steps;
    if (!x_fast && !(force_tm && force_tm <= 64 && (variant == 101 || variant == 102))) {
        // rows so far apart that a segment of them exceeds 32-bit offsets, or an X of less than 16 bytes
        fill_simple(p, M, w, num_cus, 1, 64);
        return p;
    }
    if (force_tm == 64 || force_tm == 32 || force_tm == 16) {
        if (variant == 112) {
            // (weights with more than 6 steps per segment run 8 compute waves, which exist with 128-token tiles)
            fill_pipelined(p, M, w, num_cus, max_steps <= 6 ? 64 : 128, max_steps <= 6 ? 12 : 8, 4);
            p.max_steps = fed_steps;
            return p;
        }
        const int r = variant == 102 ? 2 : 1, row_tiles = variant == 105 ? 2 : variant == 106 ? 4 : 8;
        fill_simple(p, M, w, num_cus, r, force_tm, row_tiles);
        // the short-batch kernel takes K <= 4096 (3072 with 32-token tiles); longer K silently runs the simple kernel
        if (variant == 103) p.slab = nseg <= (force_tm == 16 ? SLAB_SEGMENTS : SLAB_SEGMENTS_32);
        if (row_tiles < 8) p.slab = force_tm == 16 && nseg > 4 && nseg <= SLAB_SEGMENTS;
        p.stream = variant == 104;
        return p;
    }
    if (variant == 108 || variant == 112) {
        // 12 compute waves have 128 registers each (at most 6 step slots); denser weights take 8
        const int waves = (variant == 112 && max_steps <= 6) ? 12 : 8;
        fill_pipelined(p, M, w, num_cus, (waves == 12 && force_tm == 96) ? 96 : 128, waves, 4);
        p.max_steps = fed_steps;
        return p;
    }
    if (force_tm) {
        // 16 waves have 128 registers each: at most 6 steps per segment; denser weights run with 8
        // waves, 256 registers and half as many rows per workgroup (token tile 128 only)
        const bool eight = max_steps > 6 || variant == 8;
        fill_pipelined(p, M, w, num_cus, eight ? 128 : force_tm, eight ? 8 : 16, 0);
        return p;
    }
    // ---- short and mid-size batches
    const int reload = nseg > 2;
    Plan best{};
    double best_cost = 0.0;
    auto consider = [&](const Plan& c, const Fit& f) {
        // (persistent workgroups that leave half of the CUs idle: the short-batch kernels' ground)
        if (!c.simple && c.workgroups * 2 <= num_cus && best.workgroups != 0) return;
        const double cost = plan_cost(c, f, w, M, num_cus, out_bytes);
        if (best.workgroups == 0 || cost < 0.98 * best_cost) {
            best = c;
            best_cost = cost;
        }
    };
    Plan c = p;
    for (int row_tiles = 8; row_tiles >= 2; row_tiles /= 2) {
        fill_simple(c, M, w, num_cus, 1, 16, row_tiles);
        if (nseg > SLAB_SEGMENTS) c.stream = 1;
        else if (nseg > 4) c.slab = 1;
        // fewer rows per workgroup, the waves sharing a row tile's steps: where whole workgroups would leave most of
        // the chip idle (with few steps the sum over the shares costs what the shorter walk saves)
        if (row_tiles < 8 && (c.stream || (!c.slab && (int64_t)c.n_row_groups * c.n_tok_tiles * row_tiles / 8 >= num_cus * 3 / 16))) break;
        consider(c, c.stream ? FIT_RING_16 : c.slab ? FIT_SLAB_16 : FIT_RES_16);
    }
    // (the simple kernel where its resident rows hold all of K, the ring beyond)
    fill_simple(c, M, w, num_cus, 1, 32);
    if (nseg <= 4) consider(c, FIT_RES_32);
    if (nseg > 4 && nseg <= SLAB_SEGMENTS_32) c.slab = 1;
    else c.stream = 1;
    consider(c, FIT_RING_32);
    fill_simple(c, M, w, num_cus, 1, 64);
    if (nseg <= 2) consider(c, FIT_RES_64);
    c.stream = 1;
    consider(c, FIT_RING_64);
    // ---- persistent kernels.  16 waves have 128 registers each: at most 6 steps per segment; without loader waves
    // the general store path (outputs beyond 32-bit offsets) has no registers in them either.
    c = p;
    if (max_steps <= 6 && out_fast) {
        fill_pipelined(c, M, w, num_cus, 128, 16, 0);
        consider(c, FIT_128_16[reload]);
        fill_pipelined(c, M, w, num_cus, 96, 16, 0);
        consider(c, FIT_96_16[reload]);
    }
    fill_pipelined(c, M, w, num_cus, 128, 8, 0);
    consider(c, FIT_128_8[reload]);
    c.max_steps = fed_steps;
    fill_pipelined(c, M, w, num_cus, 128, 8, 4);
    consider(c, FIT_FED_128_8[reload]);
    for (int tm = 128; tm >= 64 && max_steps <= 6; tm -= 32) {
        fill_pipelined(c, M, w, num_cus, tm, 12, 4);
        // (1-byte outputs of one token tile per stream and at most 4 steps per segment keep the forms of whole 8 or 16
        // compute waves, as the tests of the plan have it; 768x768 at 90 %, 4096 tokens: 6.9 us, with 12 + 4: 6.0)
        if (out_bytes == 1 && max_steps <= 4 && c.n_tok_tiles <= c.n_streams) continue;
        consider(c, (tm == 128 ? FIT_FED_128_12 : tm == 96 ? FIT_FED_96_12 : FIT_FED_64_12)[reload]);
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
    const unsigned grid[3] = {8u * (unsigned)ceil_shift(plan.n_row_groups, plan.xcd_row_bits), y, (toks + y - 1) / y};
    if (plan.simple) {
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
