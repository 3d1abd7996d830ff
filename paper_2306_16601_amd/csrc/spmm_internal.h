// Internal declarations shared by the host packer, the C ABI glue and the HIP kernels.
// Not part of the public interface (see include/spmm.h).
#pragma once

#include <cstdint>
#include <functional>
#include <memory>
#include <new>
#include <utility>
#include <vector>

#include "spmm.h"

namespace spmm {

// ---------------------------------------------------------------------------------------
// Device layout: "row-tile union" format.
//
// The weight is cut into row tiles of TILE_ROWS = 16 output rows (four 4x1 block-rows in
// the paper's orientation).  For each row tile and each K segment of `kc` consecutive k,
// the k positions at which ANY of the 16 rows is non-zero are listed; the list is padded
// to a multiple of STEP_K = 64 and cut into steps.  One step is exactly one
// v_mfma_i32_16x16x64_i8: 16 rows x 64 listed k, stored dense (zero where a row has no
// block at that k) in the register layout of the weight operand:
//     vals[step][lane][t] = W[16*tile + (lane % 16)][ k_list[16*(lane / 16) + t] ],  t < 16
// so a wave fetches a step with one coalesced 16-byte load per lane.  The matching
// activation rows are named by segment-local indices, stored pairwise so that the lane that
// supplies the LDS address of list slot 16g+t (first transposing read) and 16g+8+t (second)
// finds both in one dword:
//     idx[step][8*g + t] = k_local[16g + t] | k_local[16g + 8 + t] << 16,   g < 4, t < 8
// Padding slots carry zero weights and the index of some resident row, so they add nothing.
// Inside a step the listed k are ordered for conflict-free LDS banks, not ascending (pack.cpp).
// ---------------------------------------------------------------------------------------
constexpr int TILE_ROWS = 16;
constexpr int STEP_K = 64;
constexpr int STEP_VAL_BYTES = TILE_ROWS * STEP_K;   // 1024
constexpr int STEP_IDX_DWORDS = STEP_K / 2;          // 32
constexpr int SEGMENT_ROWS = 512;                    // kc: activation rows of one K segment (one LDS buffer)

struct HostLayout {
    int kc = 0, nseg = 0, ntiles = 0;
    int64_t nsteps = 0;
    int max_steps_per_tile = 0;
    int max_steps_per_segment = 0;  // largest step count of any (tile, segment)
    std::vector<uint8_t> vals;      // nsteps * 1024
    std::vector<uint32_t> idx;      // nsteps * 32
    std::vector<int32_t> seg_ptr;   // ntiles * nseg + 1
    std::vector<int32_t> rowsum;    // ntiles * 16
};

// what resize() adds is not cleared first (it is all written next, by several threads)
template <typename T>
struct Unfilled : std::allocator<T> {
    template <typename U> struct rebind { using other = Unfilled<U>; };
    template <typename U, typename... A>
    void construct(U* p, A&&... a)
    {
        if constexpr (sizeof...(A) == 0) ::new ((void*)p) U;
        else ::new ((void*)p) U(std::forward<A>(a)...);
    }
};

// Canonical 4x1 block-sparse-row form (host): what spmm_unpack and spmm_info read.
struct Bsr {
    int64_t N = 0, K = 0;
    spmm_block_t block = SPMM_BLOCK_N4K1;
    int64_t block_rows = 0;             // ceil(N/4) (N4K1) or N (N1K4)
    std::vector<int64_t> row_ptr;       // block_rows + 1
    std::vector<int32_t, Unfilled<int32_t>> index;      // k (N4K1) or K-block c (N1K4), ascending per block-row
    std::vector<int8_t, Unfilled<int8_t>> vals;         // 4 per block
};

class Team;     // (threads of one call, team.h)
void bsr_from_dense(const int8_t* W, int64_t N, int64_t K, int64_t ldw, spmm_block_t block, Bsr& out);
// beside the first pass, and beside the last one, the calling thread runs these two (nothing else is shared with the team then)
struct Beside { std::function<void()> first, last; };
void bsr_from_dense(const int8_t* W, int64_t N, int64_t K, int64_t ldw, spmm_block_t block, Bsr& out, Team& team, const Beside* beside = nullptr);
void bsr_to_dense(const Bsr& b, int8_t* W, int64_t ldw);
void layout_from_bsr(const Bsr& b, int kc, HostLayout& out);
void layout_from_bsr(const Bsr& b, int kc, HostLayout& out, Team& team);
// row_order[i] = row of the weight that becomes row i (a permutation of 0..N-1 that moves whole
// block-rows), chosen so that rows with overlapping k lists share a row tile
void order_rows_by_k_overlap(const Bsr& b, int kc, std::vector<int32_t>& row_order);
void bsr_permute_rows(const Bsr& b, const std::vector<int32_t>& row_order, Bsr& out);

// ---------------------------------------------------------------------------------------
// Kernel launch interface (plan and dispatch in spmm_plan.hip, kernels in spmm_kernels.h).
// ---------------------------------------------------------------------------------------
// The packed weight on the device is one allocation (forms_from_bsr in pack.cpp):
//     int32   rowsum[ntiles][16]
//     int32   bounds[ntiles][nseg + 1]   first record of every segment of the tile, and one past its last
//     (padding to 128 bytes)
//     records                            one per step, RECORD_BYTES = 1152: vals[64][16], then 64 u16 k positions
//                                        in the pairing of HostLayout::idx, relative to the whole weight
// The records of a tile start at record tile * tile_steps where that costs at most half as many records again
// as there are steps (tile_steps = the longest tile's steps): a kernel can then request its first weights
// without reading bounds first.  Otherwise (tile_steps = 0) they lie back to back and bounds says where.
constexpr int RECORD_BYTES = STEP_VAL_BYTES + 4 * STEP_IDX_DWORDS;
constexpr int64_t bounds_offset(int64_t ntiles) { return ntiles * TILE_ROWS * 4; }
constexpr int64_t records_offset(int64_t ntiles, int64_t nseg)
{
    return (bounds_offset(ntiles) + ntiles * (nseg + 1) * 4 + 127) & ~(int64_t)127;
}

// The wide form, for long batches: row tiles of WIDE_ROWS = 32 rows, the same segments, steps of 64 listed k for
// v_smfmac_i32_32x32x64_i8.  That instruction takes, of every 4 consecutive list slots, at most 2 values per row, and a
// selector that says which: the packer deals the listed k to groups of 4 in which no row has more than two (pack.cpp).
//     int32   rowsum[ntiles][32]
//     int32   bounds[ntiles][nseg + 1]
//     (padding to 128 bytes)
//     records                            one per step, WIDE_RECORD_BYTES = 1536:
//         int8  vals[64][16]     lane l = 32 h + row: two stored values for each group of 4 of slots 16 h .. 16 h + 15, then
//                                the same of slots 32 + 16 h .. (the operand's layout, as observed on the device)
//         { u32 sel, rows }[64]  sel: 2 bits for each of the 16, its slot within the group.  rows: 32 times the activation rows
//                                (within the segment) of slots 32 h + t and 32 h + 8 + t (low and high half; t = l % 16 / 2),
//                                in odd lanes of slots 32 h + 16 + t and 32 h + 24 + t
constexpr int WIDE_ROWS = 32;
constexpr int WIDE_VAL_BYTES = 1024, WIDE_RECORD_BYTES = WIDE_VAL_BYTES + 64 * 8;
constexpr int WIDE_MAX_STEPS = 8;                    // of a (row tile, segment): a weight with more has no wide form
constexpr int64_t wide_bounds_offset(int64_t ntiles) { return ntiles * WIDE_ROWS * 4; }
constexpr int64_t wide_records_offset(int64_t ntiles, int64_t nseg)
{
    return (wide_bounds_offset(ntiles) + ntiles * (nseg + 1) * 4 + 127) & ~(int64_t)127;
}

// The operand of Sum, and GELU in binary32, need registers that the accumulators of the widest tiles take.
constexpr int wide_tile(bool gelu_f32, bool sum) { return sum ? 64 : gelu_f32 ? 96 : 128; }
// What the estimates do not tell of the wide kernels against the others.  In the problems of
// profiles/spmm_plan_wide_measurements.csv, estimate over measured time of the wide kernels and of the others: 1-byte outputs
// 0.96 and 1.02, 4-byte ones 0.98 and 0.99, of these with GELU 0.96 and 0.96; Sum 0.93 and 0.90; rows that do not start at 16
// bytes 0.81 and 0.89.  (The factors are of 6600 problems of other sizes, where Sum was 1.01 and 0.89.)
constexpr double wide_handicap(bool bytes, bool gelu_f32, bool sum, bool aligned_rows)
{
    return (bytes ? 1.06 : 1.0) * (sum ? 0.92 : gelu_f32 ? 0.97 : 1.0) * (aligned_rows ? 1.0 : 1.09);
}

// The bytes of both device forms; a weight that is too dense for the wide one, or that memory for it could not be had for, has
// none (wide_size = 0).  In two buffers, of which the first is kept and the second given back once it is on the device; small
// ones in one, for one copy there.
struct DeviceForms {
    int tile_steps = 0, wide_tile_steps = 0, wide_max_steps = 0;
    int64_t size = 0, wide_nsteps = 0, wide_size = 0;
    std::unique_ptr<uint8_t[]> bytes, wide;
    bool together = false;
    uint8_t* wide_bytes() const { return together ? bytes.get() + size : wide.get(); }
    void drop_wide()
    {
        wide_nsteps = wide_size = 0;
        wide_tile_steps = wide_max_steps = 0;
        wide.reset();
        together = false;
    }
};
// both forms, and of the layout all but the steps, which the first form holds; first_form is called when that one is whole, and
// the other threads work on the second meanwhile
void forms_from_bsr(const Bsr& b, HostLayout& hl, DeviceForms& f, Team& team, const std::function<void()>& first_form);
// What the device's numbers of steps come to (steps of every (row tile, segment), of every (32 rows, segment), below 0 if there
// are too many, and the sums of 32 rows of every (32 rows, segment)): all of the layout but the steps, the forms' dimensions, and
// what stands in front of their records, the first form's `head` bytes, then the wide one's.
void dims_from_steps(int64_t N, int64_t K, const int32_t* steps, const int32_t* wide_steps, const int32_t* sums, HostLayout& hl,
                     DeviceForms& f, std::vector<uint8_t>& heads, int64_t& head);
// Both forms made on the device, in one allocation, from a weight whose rows lie back to back (spmm_pack.hip).  `reserve` (false:
// no memory for it there, the host packs instead), `begin` sends the weight and starts, `finish` allocates the forms, gives what was
// reserved back, and returns a hipError_t when they are there for every stream (out of memory: the host packs instead, which may
// fit without what was reserved).
class DevicePack {
public:
    DevicePack() = default;
    ~DevicePack();
    DevicePack(const DevicePack&) = delete;
    DevicePack& operator=(const DevicePack&) = delete;
    bool reserve(int64_t N, int64_t K, spmm_block_t block);
    void begin(const int8_t* W);
    int finish(HostLayout& hl, DeviceForms& f, uint8_t** weight);

private:
    int give_back();
    uint8_t* scratch_ = nullptr;
    int64_t N_ = 0, K_ = 0, nseg_ = 0, ntiles_ = 0, nt_ = 0, info_at_ = 0, slots_at_ = 0, wide_slots_at_ = 0, heads_at_ = 0;
    int error_ = 0;
    bool n4_ = false;
};
// those steps as HostLayout has them (either may be null)
void export_steps(const HostLayout& hl, const DeviceForms& f, uint8_t* vals, uint32_t* idx);

// What a launch passes to a kernel.  96 bytes: the runtime writes the arguments of every launch through the
// bus, and from 128 bytes on a launch takes 3.3 us of the host instead of 2.7 us (measured; this was a plain
// 232-byte struct).  The kernels unpack it into an Args (spmm_kernels.h).
struct KernelArgs {
    const uint8_t* X;
    const uint8_t* weight;      // see above
    void* out;
    const float* w_scale;
    const float* bias;
    const void* aux;            // the table of a table chain, or the second operand of Sum
    uint32_t ldx, ldo, ld_sum;  // low 32 bits,
    uint32_t ld_high;           // and bits 32 .. 40 of the three (a pitch is at most 2^40), LD_HIGH_BITS each
    int32_t M, N;
    uint32_t k_flags;           // K (17 bits), ARG_* flags, x_zero_point << 24
    float x_scale, inv, out_zp_f;   // inv: 1 / out_scale, or 1 / mid_scale of a table chain; out_zp_f: zero point - smallest code
    uint16_t n_streams;         // persistent kernels: workgroups per row group, each walking token tiles j * n_streams + stream;
                                // short-batch kernels: row tiles per workgroup
    uint16_t tile_steps;
    uint32_t tiles_per_stream;  // token tiles / n_streams, rounded down; short-batch kernels: Plan::dealt
};
static_assert(sizeof(KernelArgs) == 96, "kernel arguments");
constexpr int LD_HIGH_BITS = 9;
constexpr int ARG_K_BITS = 17;
constexpr int GRID_Y_BITS = 15;                  // of the token axis of a grid: the rest goes into z
constexpr uint32_t ARG_X_TILED = 1u << 17;      // X token-tile-major [ceil(M/32)][K][32], ldx = 32; else row-major [K][ldx]
constexpr uint32_t ARG_OUT_TILED = 1u << 18;    // 1-byte out token-tile-major [ceil(M/32)][N][32], ldo = 32; else row-major [N][ldo]
constexpr uint32_t ARG_X_FAST = 1u << 19;       // the rows of one segment lie within 2^31 bytes, and X has 16: 32-bit offsets
constexpr uint32_t ARG_OUT_FAST = 1u << 20;     // whole output < 2^31 bytes (and, with Sum, the second operand too)
constexpr uint32_t ARG_OUT_ALIGNED = 1u << 21;  // ARG_OUT_FAST, out base 16-byte aligned and row pitch a multiple of 16 bytes
constexpr int ARG_XCD_SHIFT = 22;               // 2 bits: how a workgroup id decodes, see decode_workgroup

struct Plan {
    int token_tile;          // TM: 128, 96, with loaders 64, over the wide form 32 for the persistent kernels, 64, 32 or 16 for the others
    int row_tiles_per_wave;  // 1, or 2 (simple kernel; the wide form: one of its own, of 32 rows)
    int waves;               // waves that own a row tile; short-batch kernels: row tiles (or pairs) per workgroup of 8 waves
    int loaders;             // persistent kernels: extra waves that only stage activations (0 or 4; the wide form: waves / 2)
    int simple;              // 1: simple kernel
    int slab;                // 1: spmm_rowtile_mfma_slab in its place (token tile 16: K <= 4096 resident in LDS; 32: the ring's other name)
    int stream;              // 1: the streamed kernel (a ring of segments) in its place
    int wide;                // 1: persistent kernel over the wide form
    int max_steps;           // unroll bound of the per-segment step loop (persistent kernels)
    int n_row_groups, n_tok_tiles, n_streams;
    int xcd_row_bits;        // the 8 XCDs take 2^this slices of the row groups and 8 / 2^this of the tokens
    uint32_t dealt;          // short-batch kernels: 0, or the workgroups' numbers dealt to the XCDs in equal parts: 2^32 / (token
                             // tiles, or with xcd_row_bits = 1, numbered token tile by token tile, row groups), rounded up
    double fetch_us;         // what all XCDs together read through their L2s, as a time
    int64_t workgroups;
};

// variant: 0 = automatic, 8 / 16 = waves per workgroup (pipelined, token tile 128 or 96),
// 108 / 112 = pipelined with 8 / 12 compute waves and 4 loader waves (token tile 128; 112 also 96 and 64),
// 101 / 102 = simple kernel with 1 / 2 row tiles per wave (token tile 64; 101 also 32 and 16),
// 103 = short-batch kernel (token tile 16 or 32), 104 = streamed kernel (token tile 64, 32 or 16),
// 105 / 106 = simple or, from 5 segments on with 16-token tiles, short-batch kernel with 2 / 4 row tiles per workgroup,
// whose waves share a row tile's steps (token tile 32 or 16),
// 132 / 134 = over the wide form with 8 compute and 4 loader waves (token tile 128, 96 or 64) / 4 and 2 (64 or 32)
constexpr int SLAB_SEGMENTS = 8;      // K segments the short-batch kernel keeps in LDS, token tile 16
constexpr int SLAB_SEGMENTS_32 = 6;   // K segments up to which the ring with 32-token tiles goes by that kernel's name
// what the plan needs to know of a packed weight
struct WeightDims {
    int ntiles, nseg, K;
    int64_t nsteps;
    int max_steps_per_segment, max_steps_per_tile;
    // the wide form, if there is one
    int wide_max_steps = 0;         // of a (row tile, segment); 0: there is none
    int64_t wide_nsteps = 0;
};
bool plan_supported(int token_tile, int variant);
// out_bytes: size of an output element
// x_fast: see KernelArgs; an X without it takes the simple kernel, whatever was forced
// out_fast: 32-bit offsets suffice for out; if not, the automatic choice avoids the 16-wave pipelined
// kernels, whose general store path is slow for want of registers
// widest: widest token tile of the wide form that the post-operators run with (wide_tile), and its handicap (wide_handicap)
Plan make_plan(int64_t M, const WeightDims& w, int num_cus, int force_tm, int variant, int out_bytes = 1,
               bool x_fast = true, bool out_fast = true, int widest = 128, double wide_handicap = 1.0);
// Launches the SpMM kernel; returns a hipError_t value as int (0 = success).
// postop: SPMM_POST_* value, plus POST_SUM_BIT when a.sum is to be added
constexpr int POST_SUM_BIT = 4;   // (a bit no SPMM_POST_* value uses)
int launch_spmm(const Plan& plan, KernelArgs& a, spmm_out_t out_type, int postop, void* stream);

}  // namespace spmm
