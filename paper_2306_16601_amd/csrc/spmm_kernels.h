// HIP kernels for gfx950 (MI355X): 4x1 structured-sparse INT8 SpMM with fused epilogue.
//
// What the paper's Algorithm 1 does with AVX-512 (broadcast the non-zero weight words,
// re-structure the input rows named by the weight's mask into the multiply instruction's
// operand format, multiply-accumulate u8 x s8 into s32, then "downconvert" with the fused
// post-operators) is mapped to CDNA4 as follows:
//
//  * multiply instruction: v_mfma_i32_16x16x64_i8.  A row tile of 16 output rows (four 4x1
//    block-rows) is multiplied against the union of its k positions, 64 listed k per
//    instruction (layout in spmm_internal.h).
//  * "re-structure the input by the mask" (the permute/shuffle sequence of Algorithm 1):
//    the activations of one token tile and one K segment sit in LDS row-major; the
//    gathered, k-contiguous operand is produced by ds_read_b64_tr_b8, whose lanes each
//    supply the address of an arbitrary activation row -- the gather by non-zero index and
//    the byte transpose happen in the LDS read itself, no VALU shuffles.
//  * u8 x s8: the matrix instruction multiplies signed bytes, so activations are stored in
//    LDS as x - 128 (one xor per dword while staging) and 128 * rowsum(W) is added back
//    by initialising the accumulators with it; exact in int32.
//  * post-operators (Section 3.3) are applied to the accumulators in registers; the
//    GELU->int8 chain is the 256-entry table of Algorithm 2, held in LDS.
//  * the two-dimensional blocking over output rows and tokens of Section 3.2 becomes the
//    workgroup decomposition: a workgroup owns a group of row tiles and walks over token
//    tiles, so the compressed weights it needs stay in registers.
//
// Four kernels share the layout and the inner step (two transposing LDS reads, one matrix
// instruction per 16 tokens), a fifth (spmm_wide.h) has a layout of its own; the host's plan
// (spmm_plan.hip) picks one by its estimate of their times:
//   spmm_rowtile_mfma         persistent, software-pipelined: long batches
//   spmm_rowtile_mfma_fed     the same with waves that only stage activations: long batches with 4-byte
//                             outputs, weights that do not stay in registers, or rows that 12 waves divide better
//   spmm_rowtile_mfma_simple  one workgroup per 32 to 128 rows x 16/32/64 tokens, the whole K slab (up to
//                             2048 rows at a time, 1024 with 64 tokens) in LDS at once: small problems.
//                             spmm_rowtile_mfma_slab<16> is the same with 4096 resident rows
//   spmm_rowtile_mfma_stream  a ring of four segments of activations: mid-size batches, short ones with the longest K.
//                             spmm_rowtile_mfma_slab<32> is the same code under the name by which the plan reports
//                             32-token tiles of 5 to 6 segments
//   spmm_rowtile_smfmac       persistent, 32-row tiles on the structured-sparse instruction: long batches of weights
//                             that have that form
//
// Lane roles of the matrix instruction (D = A.B, 64 lanes, g = lane / 16, c = lane % 16):
//   A operand (activations): row = token c, bytes t = k-list slots 16g .. 16g+15
//   B operand (weights)    : column = output row c, same k slots
//   D                      : D[token 4g + r][output row c], r = 0..3
//
// ds_read_b64_tr_b8 within a 16-lane group: the lane at position p supplies the address of
// 8 bytes; result lane p receives, as byte t, byte (p % 8) of the 8 bytes addressed by
// source position 2t + p / 8.  With source position 2t + h pointing at tokens 8h .. 8h+7
// of activation row k_t, result lane p holds token p of rows k_0 .. k_7.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "spmm_internal.h"

namespace spmm {

// KernelArgs, unpacked: what the kernels work with (scalar registers; what a kernel does not use costs nothing)
struct Args {
    const uint8_t* records;     // step records of the packed weight
    const int32_t* bounds;      // [ntiles][nseg + 1]
    const int32_t* rowsum;
    const uint8_t* X;
    void* out;
    const float* w_scale;
    const float* bias;
    const int8_t* lut;
    const float* sum;           // Sum post-operator: [N][ld_sum]
    int64_t ldx, ldo, ld_sum;
    int64_t x_last16;           // offset of the last 16 bytes of X: no 16-byte read goes beyond them (negative: X has fewer)
    int N, K, M, nseg, ntiles, tile_steps;
    int n_streams, tiles_per_stream;   // persistent kernels
    int wg_tiles;               // short-batch kernels: row tiles (or pairs of them) per workgroup
    uint32_t dealt;             // short-batch kernels: see decode_tile
    int xcd_row_bits;           // the 8 XCDs take 2^this slices of the row groups x 8 / 2^this slices of the tokens
    int corr_mul;               // 128 - x_zero_point: the activations are multiplied as (x - 128)
    float x_scale, inv, out_zp_f;
    bool x_fast, out_fast, out_aligned;
    int x_tile_stride;          // token-tile-major X: bytes between tiles, 32 K; else 0
    int out_tile_stride;        // token-tile-major output: 32 N; else 0
    uint32_t out_bytes;         // with out_fast: bytes from out to the end of the last element the call may write
};

template <int OUT>
__device__ __forceinline__ Args unpack(const KernelArgs& p)
{
    Args a;
    a.M = p.M;
    a.N = p.N;
    a.K = (int)(p.k_flags & ((1u << ARG_K_BITS) - 1));
    a.nseg = (a.K + SEGMENT_ROWS - 1) / SEGMENT_ROWS;
    a.ntiles = (a.N + TILE_ROWS - 1) / TILE_ROWS;
    a.tile_steps = p.tile_steps;
    a.rowsum = (const int32_t*)p.weight;
    a.bounds = (const int32_t*)(p.weight + bounds_offset(a.ntiles));
    a.records = p.weight + records_offset(a.ntiles, a.nseg);
    a.X = p.X;
    a.out = p.out;
    a.w_scale = p.w_scale;
    a.bias = p.bias;
    a.lut = (const int8_t*)p.aux;
    a.sum = (const float*)p.aux;
    constexpr uint32_t high = (1u << LD_HIGH_BITS) - 1;
    a.ldx = (int64_t)((uint64_t)p.ldx | (uint64_t)(p.ld_high & high) << 32);
    a.ldo = (int64_t)((uint64_t)p.ldo | (uint64_t)(p.ld_high >> LD_HIGH_BITS & high) << 32);
    a.ld_sum = (int64_t)((uint64_t)p.ld_sum | (uint64_t)(p.ld_high >> 2 * LD_HIGH_BITS & high) << 32);
    const int tiles32 = (a.M + SPMM_X_TILE - 1) / SPMM_X_TILE;
    const bool xt = p.k_flags & ARG_X_TILED, ot = p.k_flags & ARG_OUT_TILED;
    a.x_tile_stride = xt ? a.K * SPMM_X_TILE : 0;
    a.out_tile_stride = ot ? a.N * SPMM_X_TILE : 0;
    a.x_last16 = xt ? (int64_t)tiles32 * a.x_tile_stride - 16 : (int64_t)(a.K - 1) * a.ldx + a.M - 16;
    a.out_bytes = ot ? (uint32_t)tiles32 * (uint32_t)a.out_tile_stride
                     : ((uint32_t)(a.N - 1) * p.ldo + (uint32_t)a.M) * (OUT == SPMM_OUT_S32 || OUT == SPMM_OUT_F32 ? 4u : 1u);
    a.x_fast = p.k_flags & ARG_X_FAST;
    a.out_fast = p.k_flags & ARG_OUT_FAST;
    a.out_aligned = p.k_flags & ARG_OUT_ALIGNED;
    a.xcd_row_bits = (int)(p.k_flags >> ARG_XCD_SHIFT & 3);
    a.corr_mul = 128 - (int)(p.k_flags >> 24);
    a.x_scale = p.x_scale;
    a.inv = p.inv;
    a.out_zp_f = p.out_zp_f;
    a.n_streams = p.n_streams;
    a.wg_tiles = p.n_streams;
    a.tiles_per_stream = (int)p.tiles_per_stream;
    a.dealt = p.tiles_per_stream;
    return a;
}

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v2i* lds_v2i_ptr;

// The same vectors at any address: global memory takes 16-byte (and dword) accesses at byte alignment on
// this hardware (LLVM's unaligned-access-mode, on for the HSA target), so an unpadded row pitch costs the
// cache lines that a piece straddles and nothing else.
struct __attribute__((packed)) v4i_any { v4i v; };
struct __attribute__((packed)) v4f_any { v4f v; };
struct __attribute__((packed)) u32_any { uint32_t v; };
struct __attribute__((packed)) v2i_any { v2i v; };
struct __attribute__((packed)) u16_any { uint16_t v; };
__device__ __forceinline__ v4i load16_any(const void* p) { return ((const v4i_any*)p)->v; }

// v, as a value the compiler knows nothing of: what is worked out from it is worked out where it stands, and not ahead
// of the phase loop of a persistent kernel, where it would occupy registers throughout.  The 16-wave kernels have 128
// and need them: with addresses, columns and rows kept across the phases up to 20 were spilled, weight rows among them,
// and a spilled load is waited for as soon as it is issued, with every load before it.  Measured, kept -> worked out
// (6144 tokens, table chain, tile-major, 80 %): 1024 x 1024 11.2 -> 9.7 us, 4096 x 1024 27.8 -> 26.4; 1024 x 4096 with
// Sum, int8 31.7 -> 29.7; 1024 x 1024 with Sum, binary32 rows 18.5 -> 16.6.
template <typename T>
__device__ __forceinline__ T pinned(T v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// The same for a loop over `turn`, a uniform value that changes with every turn.  (pinned counts as a write to memory: what a
// uniform address is read for after it comes through vector loads, not scalar ones.)
template <typename T>
__device__ __forceinline__ T pinned_in_turn(T v, const int turn)
{
    asm("" : "+v"(v) : "s"(turn));
    return v;
}

constexpr int FLIP = (int)0x80808080;   // x ^ 0x80 == x - 128 as a signed byte

// GELU in its erf form, y * Phi(y) = 0.5 * y * erfc(-y / sqrt(2)), in binary32, branch-free.
// With z = |y| / sqrt(2) and t = 2 / (2 + z), ln(erfc(z) exp(z^2) / t) is smooth on 0 < t <= 1
// (it tends to -ln(2 sqrt(pi)) as z grows), so erfc(z) = t * exp(P(t) - z^2) with P a degree-9
// polynomial: a least-squares fit of that function at 400 Chebyshev nodes, converted to powers
// of t.  The negative side is 0.5 * y * erfc(z) and keeps its relative accuracy in the tail; the
// positive side is y - 0.5 * y * erfc(z).  The rounding of z^2 and of the exponent grows with z^2,
// to about 2e-6 relative at |y| = 5; beyond |y| = 3 the result is below 4.1e-3 and the absolute
// part of the tolerance (1e-7) covers it.  Measured against the exact value on a dense sweep the
// error stays below a tenth of 1e-5 * |GELU| + 1e-7.
__device__ __forceinline__ float gelu_f32(float y)
{
    const float z = fabsf(y) * 0.70710678118654752440f;
    const float t = __builtin_amdgcn_rcpf(__fmaf_rn(0.5f, z, 1.0f));
    float p = 1.708727777e-01f;
    p = __fmaf_rn(p, t, -8.221522344e-01f);
    p = __fmaf_rn(p, t, 1.488515889e+00f);
    p = __fmaf_rn(p, t, -1.135204000e+00f);
    p = __fmaf_rn(p, t, 2.788680845e-01f);
    p = __fmaf_rn(p, t, -1.862880617e-01f);
    p = __fmaf_rn(p, t, 9.678418949e-02f);
    p = __fmaf_rn(p, t, 3.740919597e-01f);
    p = __fmaf_rn(p, t, 1.000023680e+00f);
    p = __fmaf_rn(p, t, -1.265512225e+00f);
    // exp(p - z^2) = 2^((p - z^2) * log2(e)); below 2^-126 the result flushes towards zero, where
    // |GELU| < 1e-30 anyway
    const float e = t * __builtin_amdgcn_exp2f((p - z * z) * 1.4426950408889634f);
    const float h = 0.5f * y * e;          // y < 0: the result; y >= 0: what is missing from y
    return y < 0.0f ? h : y - h;
}

// Where the table of Algorithm 2 is read from.
struct GlobalLut {
    const int8_t* p;
    __device__ __forceinline__ uint32_t operator()(uint32_t key) const { return (uint8_t)p[key]; }
};

struct LdsTable {
    static constexpr bool CONSTANTS = true;        // a register for a constant can be had where this is used
    const uint8_t* p;
    __device__ __forceinline__ uint32_t operator()(uint32_t key) const { return p[key]; }
};

// POST template parameters below are the SPMM_POST_* value, plus POST_SUM_BIT when the Sum
// post-operator (a second binary32 tensor added after BiasAdd / GeLU, before Quantize) is on.

// Output stores of the aligned paths go through a buffer resource that covers exactly the bytes
// the call may write (out_bytes, < 2 GiB on these paths): a store beyond it is dropped by the
// hardware.  Where one store instruction of a wave fills whole 128-byte lines (1-byte outputs in
// token-tile-major order: 16 rows x 32 bytes back to back) or the output is 4 bytes wide, the
// store goes out at agent scope (sc1), i.e. written through the XCD's L2 as it is issued: left at
// the default scope the lines stay dirty in that L2 and are written back when the kernel ends,
// behind all the compute, and that write-back is then the tail of every launch (measured inside
// the rotating benchmark step, outputs going to HBM: 4096 x 1024 at 90 %, 24.8 -> 23.1 us; binary32
// 3072 x 768, 18.4 -> 17.2 us).  Row-major 1-byte outputs leave in 64-byte runs, half a line per
// instruction; written through, those cost more at the memory than they save (25.0 -> 27.3 us),
// so they stay at the default scope and the L2 merges them.
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
constexpr int SCOPE_DEFAULT = 0, SCOPE_AGENT = 16;   // cache-policy operand of the buffer stores: none / sc1
__device__ __forceinline__ __amdgpu_buffer_rsrc_t out_resource(const Args& a)
{
    // raw buffer (stride 0), 32-bit data format
    return __builtin_amdgcn_make_buffer_rsrc(a.out, 0, (int)a.out_bytes, 0x00020000);
}
// (byte_off: per lane; uniform_off: the same for the whole wave, held in a scalar register)
template <int SCOPE, typename V>
__device__ __forceinline__ void store16_out(const __amdgpu_buffer_rsrc_t rs, const uint32_t byte_off, const V v,
                                            const uint32_t uniform_off = 0)
{
    static_assert(sizeof(V) == 16, "16-byte store");
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, v), rs, (int)byte_off, (int)uniform_off, SCOPE);
}

// Quantised codes of four pre-activations (Quantize post-operator / table look-up), packed.
// v_cvt_pk_u8_f32 converts with saturation to [0, 255] and puts the byte in its place, in one instruction: signed
// codes go through it with 128 added (KernelArgs::out_zp_f) and taken off the whole word.  (Clamping, converting and
// packing one by one is 3.5 instructions more per value, and the post-operators of a 96-token tile keep the vector units
// of a CU busy for as long as half a segment of multiplying does.)
// key = sat_s8(rint(v)) + 128: v is clamped, scaled so that one is the smallest denormal, and 128 of those added, rounded once,
// half to even (128 is even): the bits are the key.  Two instructions instead of the three of rounding, adding and
// v_cvt_pk_u8_f32, which take no constant but those in the instruction (1024x1024 at 90 %, 6144 tokens, GELU to s8, on one
// machine: 9.18 us, now 9.02; machines differ by as much).
template <bool CONSTANTS>
__device__ __forceinline__ uint32_t table_key(const float v)
{
    if constexpr (!CONSTANTS) return __builtin_amdgcn_cvt_pk_u8_f32(rintf(v) + 128.0f, 0u, 0u);
    return __builtin_bit_cast(uint32_t, __fmaf_rn(__builtin_amdgcn_fmed3f(v, -128.0f, 127.0f), 0x1p-149f, 0x1p-142f));
}

template <int OUT, int POST, typename Lut>
__device__ __forceinline__ uint32_t quantise4(const Args& a, const float (&y)[4], const Lut& lut)
{
    if constexpr ((POST & SPMM_POST_GELU) != 0) {
        uint32_t q[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) q[r] = lut(table_key<Lut::CONSTANTS>(y[r] * a.inv));
        return __builtin_amdgcn_perm(q[1], q[0], 0x0c0c0400u) | __builtin_amdgcn_perm(q[3], q[2], 0x04000c0cu);
    } else {
        uint32_t q = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) q = __builtin_amdgcn_cvt_pk_u8_f32(rintf(y[r] * a.inv) + a.out_zp_f, r, q);
        return OUT == SPMM_OUT_U8 ? q : q ^ (uint32_t)FLIP;
    }
}

// The second operand of Sum for tokens m0 .. m0 + 3 of output row n, m0 < M (none of it is read outside [N][M])
// TIGHT: tokens past the end repeat the first one instead of being zero (either way they are never stored): zeros
// would be kept in registers all through a persistent kernel.
template <int POST, bool TIGHT = false>
__device__ __forceinline__ v4f load_sum4(const Args& a, const int n, const int m0)
{
    v4f v = {0.0f, 0.0f, 0.0f, 0.0f};
    if constexpr ((POST & POST_SUM_BIT) != 0) {
        const float* sp = a.sum + (int64_t)n * a.ld_sum + m0;
        if (m0 + 4 <= a.M) {
            v = ((const v4f_any*)sp)->v;
        } else {
            if constexpr (TIGHT) v = (v4f){sp[0], sp[0], sp[0], sp[0]};
#pragma unroll
            for (int r = TIGHT; r < 3; ++r)
                if (m0 + r < a.M) v[r] = sp[r];
        }
    }
    return v;
}

// Generic post-operators + store for 4 consecutive tokens m0..m0+3 of output row n: any
// alignment, any tail (the slow path of every kernel).
// WIDE: 4-byte outputs whose 16-byte pieces are aligned go out at agent scope (see out_resource);
// costs registers the 16-wave pipelined kernels do not have (their full tiles take finish_tile_fast).
// OT: layout of a 1-byte output: 1 = token-tile-major, 0 = row-major, -1 = whichever the arguments say
// sum4: the operand of Sum for these tokens (load_sum4), where there is one.
template <int OUT, int POST, bool WIDE = false, int OT = -1, typename Lut>
__device__ __forceinline__ void finish4(const Args& a, const v4i acc, const float s, const float b,
                                        const int n, const int m0, const Lut& lut, const v4f sum4)
{
    const int valid = a.M - m0;   // > 0 guaranteed by caller
    if constexpr (OUT == SPMM_OUT_S32) {
        int32_t* o = (int32_t*)a.out + (int64_t)n * a.ldo + m0;
        if (WIDE && a.out_aligned && valid >= 4) {
            store16_out<SCOPE_AGENT>(out_resource(a), 4u * ((uint32_t)n * (uint32_t)a.ldo + (uint32_t)m0), acc);
        } else if (valid >= 4) {
            ((v4i_any*)o)->v = acc;
        } else {
            for (int r = 0; r < 4; ++r)
                if (r < valid) o[r] = acc[r];
        }
    } else {
        float y[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) y[r] = __fmaf_rn((float)acc[r], s, b);
        if constexpr (OUT == SPMM_OUT_F32 && (POST & SPMM_POST_GELU) != 0) {
#pragma unroll
            for (int r = 0; r < 4; ++r) y[r] = gelu_f32(y[r]);
        }
        if constexpr ((POST & POST_SUM_BIT) != 0) {
#pragma unroll
            for (int r = 0; r < 4; ++r) y[r] = y[r] + sum4[r];
        }
        if constexpr (OUT == SPMM_OUT_F32) {
            float* o = (float*)a.out + (int64_t)n * a.ldo + m0;
            const v4f v = {y[0], y[1], y[2], y[3]};
            if (WIDE && a.out_aligned && valid >= 4) {
                store16_out<SCOPE_AGENT>(out_resource(a), 4u * ((uint32_t)n * (uint32_t)a.ldo + (uint32_t)m0), v);
            } else if (valid >= 4) {
                ((v4f_any*)o)->v = v;
            } else {
                for (int r = 0; r < 4; ++r)
                    if (r < valid) o[r] = y[r];
            }
        } else {
            const uint32_t q = quantise4<OUT, POST>(a, y, lut);
            // (token-tile-major output, [M / 32][N][32]: rows 32 bytes apart, a column's tile out_tile_stride
            // = 32 N bytes after the previous one; four consecutive tokens from a multiple of 4 share a tile)
            const bool ot = (OT == 1) || (OT == -1 && a.out_tile_stride != 0);
            uint8_t* o = (uint8_t*)a.out + (int64_t)n * a.ldo +
                         (ot ? (int64_t)(m0 >> 5) * a.out_tile_stride + (m0 & 31) : (int64_t)m0);
            if (valid >= 4) {
                ((u32_any*)o)->v = q;
            } else {
                for (int r = 0; r < 4; ++r)
                    if (r < valid) o[r] = (uint8_t)(q >> 8 * r);
            }
        }
    }
}

// One step's weight operand and this lane's pair of activation rows from the step records; `step` is the same
// for the whole wave.  (The rows are positions in the whole weight; they are cut to the segment where they are
// used, first_row / second_row, and not here, where it would mean waiting for the load.)
__device__ __forceinline__ void load_step(const Args& a, const int step, const int lane, v4i& w, uint32_t& rows)
{
    const uint8_t* r = a.records + (int64_t)step * RECORD_BYTES;
    w = *(const v4i*)(r + (uint32_t)lane * 16u);
    rows = *(const uint32_t*)(r + (STEP_VAL_BYTES + 32u * (uint32_t)(lane >> 4) + 4u * (uint32_t)((lane & 15) >> 1)));
}
__device__ __forceinline__ uint32_t first_row(const uint32_t rows) { return rows & (SEGMENT_ROWS - 1); }
__device__ __forceinline__ uint32_t second_row(const uint32_t rows) { return rows >> 16 & (SEGMENT_ROWS - 1); }

// s_waitcnt vmcnt(0) only (expcnt / lgkmcnt fields left at their maxima).  Issued when the
// prefetches started at the beginning of a phase have long landed: it tells the compiler's
// wait-count bookkeeping that no global load is outstanding, so the next phase's multiply
// loop does not stall on the prefetches issued just before it.
__device__ __forceinline__ void wait_global_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// Byte offset of token column `col` inside an activation row.  Row-major X: the column itself (rows
// are ldx apart).  Token-tile-major X, [ceil(M / 32)][K][32] (the re-structured input of Section 3.2:
// the rows of a 32-token tile lie back to back, so a workgroup's token tile is three or four
// contiguous regions of memory): rows are 32 bytes apart and a column's tile starts
// x_tile_stride = 32 K bytes after the previous one.  16-byte pieces start at multiples of 16 and
// never straddle two tiles; xcol(c1 + c2) = xcol(c1) + xcol(c2) when c1 is a multiple of 32.
// XT: 1 = token-tile-major, 0 = row-major, -1 = whichever the arguments say (a uniform run-time test).
// The pipelined kernel is instantiated for both layouts: its 16-wave forms have no register to spare
// for a choice at run time.
template <int XT = -1>
__device__ __forceinline__ int xcol(const Args& a, const int col)
{
    // (the whole X is smaller than 2 GiB in this layout, checked on the host: the offset fits an int)
    if constexpr (XT == 0) return col;
    else if constexpr (XT == 1) return (col >> 5) * a.x_tile_stride + (col & 31);
    else return a.x_tile_stride ? (col >> 5) * a.x_tile_stride + (col & 31) : col;
}

// 16-byte pieces of one segment's activation rows in the token tile that is cut by the end of the rows, at
// any alignment.  Tokens from M on are never stored, so what their bytes hold does not matter: a piece
// beyond the end reads the start of its row, a piece cut by it reads on into the next row.  Only where
// those 16 bytes would leave the matrix (its last row; rows shorter than a piece) is the read moved back
// to the last 16 bytes, and the loaded piece then shifted into place.  Segments with such rows are known
// beforehand (`inside` is uniform): everywhere else nothing touches the loaded registers before they are
// used, and the loads stay in flight.  Offsets are 32 bits from a uniform base (KernelArgs::x_fast); the
// base lies 16 bytes before the segment so that a read moved back into the previous one is not negative.
template <int XT = -1>
struct RaggedPieces {
    const Args& a;
    const uint8_t* base;
    uint32_t bias, limit;
    bool inside;
    __device__ __forceinline__ RaggedPieces(const Args& args, const int k0, const int last) : a(args)
    {
        bias = k0 > 0 ? 16 : 0;
        base = a.X + ((int64_t)k0 * a.ldx - bias);
        const int64_t left = a.x_last16 - ((int64_t)k0 * a.ldx - bias);      // >= 0
        limit = left < 0x7fffffff ? (uint32_t)left : 0x7fffffffu;
        inside = a.x_tile_stride != 0 || bias + (uint32_t)last * (uint32_t)a.ldx + (uint32_t)((a.M - 1) & ~15) <= limit;
    }
    __device__ __forceinline__ uint32_t offset(const int row, const int col) const
    {
        return bias + (uint32_t)row * (uint32_t)a.ldx + (uint32_t)xcol<XT>(a, col < a.M ? col : 0);
    }
    __device__ __forceinline__ v4i load(const int row, const int col) const
    {
        return load16_any(base + min(offset(row, col), limit));
    }
    __device__ __forceinline__ v4i shifted(v4i v, const int row, const int col) const
    {
        const uint32_t off = offset(row, col), back = off - min(off, limit);      // 0 .. 15
        if (back & 8) v = (v4i){v[2], v[3], 0, 0};
        if (back & 4) v = (v4i){v[1], v[2], v[3], 0};
        v4i r;
#pragma unroll
        for (int w = 0; w < 4; ++w)
            r[w] = (int)__builtin_amdgcn_alignbyte(w < 3 ? (uint32_t)v[w + 1] : 0u, (uint32_t)v[w], back & 3);
        return r;
    }
};
// The same for a row-major matrix whose segments exceed 32-bit offsets, or that holds less than 16 bytes
// (only the simple kernel takes those, see make_plan): pieces that would leave the matrix byte by byte.
__device__ __forceinline__ v4i load_x16_far(const Args& a, const int row, const int col)
{
    const int64_t off = (int64_t)row * a.ldx + (col < a.M ? col : 0);
    if (off <= a.x_last16) return load16_any(a.X + off);
    v4i v = {0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < 16; ++j)
        if (col + j < a.M) v[j >> 2] |= (int)((uint32_t)a.X[off + j] << (8 * (j & 3)));
    return v;
}

// Workgroup id -> (row group, token tile or stream).  Workgroups go round the 8 XCDs, each with an L2 of its
// own, in linear order (x fastest, gridDim.x a multiple of 8): XCD x & 7 takes one of 2^xcd_row_bits slices of the
// row groups and one of the 8 / 2^xcd_row_bits slices of the tokens, so every XCD reads that share of the packed
// weight and of the activations through its L2 and no more (the host picks the split that reads least).
// Neighbouring token tiles stay on one XCD: tiles narrower than a cache line share their lines.
// The token axis may exceed one grid dimension: y and z.  False: a padding workgroup.
__device__ __forceinline__ bool decode_workgroup(const Args& a, const int n_row_groups, const int n_tokens, int& rg, int& tt)
{
    const int xcd = blockIdx.x & 7, rb = a.xcd_row_bits, tb = 3 - rb;
    const int rows = (n_row_groups + (1 << rb) - 1) >> rb, toks = (n_tokens + (1 << tb) - 1) >> tb;
    const int r = (int)(blockIdx.x >> 3), t = (int)(blockIdx.y + (blockIdx.z << GRID_Y_BITS));
    rg = (xcd & ((1 << rb) - 1)) * rows + r;
    tt = (xcd >> rb) * toks + t;
    return rg < n_row_groups && t < toks && tt < n_tokens;
}

// The same for the kernels of one workgroup per (row group, token tile), where slices would give some XCD more workgroups than
// it has CUs while the others have CUs left (12 row groups x 21 token tiles: 33 and 30, for 32): the workgroups are numbered
// row group by row group, or token tile by token tile (the host's choice again), and the numbers dealt out in eight equal parts.
__device__ __forceinline__ bool decode_tile(const Args& a, const int n_row_groups, const int n_tokens, int& rg, int& tt)
{
    if (!a.dealt) return decode_workgroup(a, n_row_groups, n_tokens, rg, tt);
    const uint32_t all = (uint32_t)n_row_groups * (uint32_t)n_tokens;
    const uint32_t i = (blockIdx.x & 7) * ((all + 7) >> 3) + (blockIdx.x >> 3);
    const bool by_tokens = a.xcd_row_bits != 0;
    // (dealt: 2^32 / the divisor, rounded up: exact as all < 2^16)
    const uint32_t q = (uint32_t)((uint64_t)i * a.dealt >> 32), r = i - q * (uint32_t)(by_tokens ? n_row_groups : n_tokens);
    rg = (int)(by_tokens ? r : q);
    tt = (int)(by_tokens ? q : r);
    return i < all;
}

// =======================================================================================
// Pipelined persistent kernel: long batches.  What bounds it is the LDS -- the gather reads 1 KB of it per step
// and 16 tokens at 121 bytes a clock per CU -- and then the times in which it is idle because all waves of the
// workgroup do something else together: requesting the next phase and the post-operators (4096 x 1024 at 85 %, 6144
// tokens, table chain, row-major: 24.7 us, tile-major 22.3, of which 11 us gather, 3.5 us the start, about a quarter the
// post-operators; workgroups of 8 waves, to overlap them, read X twice as often and take 31.0 us row-major).
//
// Workgroup = NW waves.  Wave w owns row tile NW*rg + w (16 output rows) for the whole
// kernel; the workgroup walks over token tiles of TM tokens (stream, stream + S, ..) and,
// inside a token tile, over the K segments of 512 rows.  One (token tile, segment) pair is a
// "phase".  LDS holds two activation buffers [512 rows][TM + 16 bytes]; while phase p
// multiplies out of buffer p % 2, the global loads for phase p+1 are in flight in registers
// and are written to the other buffer afterwards; one barrier per phase.  The compressed
// weights of a phase (at most MAXS steps of 64 listed k) live in one of two register sets;
// with at most two segments they are loaded once per workgroup and reused for every token
// tile, otherwise they are prefetched one phase ahead.
//
// Two token-tile widths, both with one workgroup per CU, the table at LDS offset 0 and the
// buffers behind it; the plan takes the one it estimates to be faster (spmm_plan.hip):
//   TM = 128: fewer phases for the same tokens.
//   TM =  96: where it divides the tokens into a number of tiles that fills the CUs more evenly
//             (1024 x 1024 at 90 %, 6144 tokens: 256 workgroups instead of 192, 8.7 us instead of 9.1,
//             tile-major 7.6 instead of 8.9).  A row is 6 pieces of 16 bytes; 3/4 of the threads stage them.
// Every LDS row has 16 spare bytes behind its TM tokens (the pitch TM + 16 makes consecutive
// rows start 4 banks apart).  These spare chunks carry the output staging for 1-byte outputs:
// wave w transposes its 16 rows x 64 tokens through chunks 64w .. 64w+63 so that a row's
// tokens leave in 64-byte runs (32 for the last third of a 96-token tile) instead of 4-byte
// pieces.  Staging row r, 16-token piece j lives in chunk 4r + (j ^ (r >> 2)): with both
// pitches the 4-byte writes and the 16-byte reads then touch every LDS bank once.
// =======================================================================================
template <int TM>
struct Geo;

template <>
struct Geo<128> {
    static constexpr int STRIDE = 144, PIECES = 8, HALVES = 2;
    static constexpr int BUF = SEGMENT_ROWS * STRIDE;   // 73728
    static constexpr int X0 = 256;                      // table in [0, 256): the key is the address
    static constexpr int LDS = X0 + 2 * BUF;
    static __device__ __forceinline__ uint32_t lut_addr(uint32_t key) { return key; }
    // spare chunk n in [0, 1024): behind row n of the two back-to-back buffers
    static __device__ __forceinline__ uint32_t chunk(uint32_t n) { return X0 + n * STRIDE + 128; }
};

template <>
struct Geo<96> {
    static constexpr int STRIDE = 112, PIECES = 6, HALVES = 2;
    static constexpr int BUF = SEGMENT_ROWS * STRIDE;   // 57344
    static constexpr int X0 = 256;
    static constexpr int LDS = X0 + 2 * BUF;
    static __device__ __forceinline__ uint32_t lut_addr(uint32_t key) { return key; }
    static __device__ __forceinline__ uint32_t chunk(uint32_t n) { return X0 + n * STRIDE + 96; }
};

// TM = 64 (loader-wave kernel only): four pieces per row, twice as many tiles per stream; the output
// stores of a workgroup then start after half the time and the last tile's burst is half as long.
// (3072 x 768 at 85 %, 4096 tokens, row-major: int8 13.1 us, 128-token tiles 13.2, 96 15.9, 16 waves without loaders 15.6;
// binary32 16.6, 16.7, 18.6 and 22.0.)
template <>
struct Geo<64> {
    static constexpr int STRIDE = 80, PIECES = 4, HALVES = 1;
    static constexpr int BUF = SEGMENT_ROWS * STRIDE;   // 40960
    static constexpr int X0 = 256;
    static constexpr int LDS = X0 + 2 * BUF;
    static __device__ __forceinline__ uint32_t lut_addr(uint32_t key) { return key; }
    static __device__ __forceinline__ uint32_t chunk(uint32_t n) { return X0 + n * STRIDE + 64; }
};

template <int TM, bool TIGHT = false>
struct LdsLut {
    static constexpr bool CONSTANTS = !TIGHT;
    const uint8_t* lds;
    __device__ __forceinline__ uint32_t operator()(uint32_t key) const { return lds[Geo<TM>::lut_addr(key)]; }
};

// Whether full token tiles go through finish_tile_fast.  4-byte outputs in rows that are not 16-byte aligned
// go through finish4: its plain stores leave the lines that a piece straddles to the L2 to merge (2304 x 768,
// 4095 tokens in rows of 4095, binary32: 26.8 us with stores at agent scope, 19.9 us at the default scope).
template <int OUT>
__device__ __forceinline__ bool takes_fast_stores(const Args& a)
{
    return (OUT == SPMM_OUT_S8 || OUT == SPMM_OUT_U8) ? a.out_fast : a.out_aligned;
}

// The first `count` of 16 bytes, 1 .. 15 of them.  (Every byte of a wave's store goes to a row of its own, 64 lines a store: one
// by one, the last tokens of a tile took as long as a third of its multiplying.  1024x1024 at 90 %, 6143 tokens, s8: 10.4 us,
// 6144 tokens 8.7.)
__device__ __forceinline__ void store_cut16(uint8_t* to, v4i v, const int count)
{
    if (count & 8) {
        ((v2i_any*)to)->v = (v2i){v[0], v[1]};
        to += 8;
        v = (v4i){v[2], v[3], 0, 0};
    }
    if (count & 4) {
        ((u32_any*)to)->v = (uint32_t)v[0];
        to += 4;
        v[0] = v[1];
    }
    if (count & 2) {
        ((u16_any*)to)->v = (uint16_t)v[0];
        to += 2;
        v[0] = (int)((uint32_t)v[0] >> 16);
    }
    if (count & 1) *to = (uint8_t)v[0];
}

// Post-operators + store for one full token tile of one wave, everything in bounds (4-byte outputs:
// and aligned): lane (g, c) holds tokens tok0 + 16 i + 4 g + {0..3} of output row 16 * tile + c.
// 4-byte outputs are stored straight from the accumulator layout (16 bytes per lane, 64-byte
// runs per row); 1-byte outputs go through the LDS staging chunks, also of a tile that the end of the tokens cuts (CUT).
// TIGHT: without a register for table_key's constants (the forms of 16 waves with 6 step slots spill one)
template <int TM, int OUT, int POST, int OT = -1, bool TIGHT = false, bool CUT = false>
__device__ __forceinline__ void finish_tile_fast(const Args& a, const v4i (&acc)[Geo<TM>::PIECES],
                                                 const float scale, const float bias, const int tile,
                                                 const int tok0, int lane, const int wave, uint8_t* lds)
{
    using G = Geo<TM>;
    lane = pinned(lane);
    const int g = lane >> 4, c = lane & 15;
    if constexpr (OUT == SPMM_OUT_S32) {
        // fast path: the whole output is < 2 GiB (checked on the host), 32-bit offsets suffice
        const uint32_t off = (uint32_t)(tile * TILE_ROWS + c) * (uint32_t)a.ldo + (uint32_t)(tok0 + 4 * g);
        const __amdgpu_buffer_rsrc_t rs = out_resource(a);
        if (tile * TILE_ROWS + c < a.N) {
#pragma unroll
            for (int i = 0; i < G::PIECES; ++i) store16_out<SCOPE_AGENT>(rs, 4u * off + 64u * i, acc[i]);
        }
    } else if constexpr (OUT == SPMM_OUT_F32) {
        const uint32_t off = (uint32_t)(tile * TILE_ROWS + c) * (uint32_t)a.ldo + (uint32_t)(tok0 + 4 * g);
        const __amdgpu_buffer_rsrc_t rs = out_resource(a);
        // (Sum: the second operand is read in the accumulator layout, 16 bytes per lane)
        const float* sp = a.sum + ((uint32_t)(tile * TILE_ROWS + c) * (uint32_t)a.ld_sum + (uint32_t)(tok0 + 4 * g));
        if (tile * TILE_ROWS + c < a.N) {
#pragma unroll
            for (int i = 0; i < G::PIECES; ++i) {
                v4f y;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    y[r] = __fmaf_rn((float)acc[i][r], scale, bias);
                    if constexpr ((POST & SPMM_POST_GELU) != 0) y[r] = gelu_f32(y[r]);
                }
                if constexpr ((POST & POST_SUM_BIT) != 0) y = y + ((const v4f_any*)(sp + 16 * i))->v;
                store16_out<SCOPE_AGENT>(rs, 4u * off + 64u * i, y);
            }
        }
    } else {
        const LdsLut<TM, TIGHT> lut{lds};
        // write side: this lane's quad of piece j goes to staging row c, piece j
        const uint32_t wbase = G::chunk(64 * wave + 4 * c) + 4 * g;
        const int wsw = c >> 2;
        // read side: this lane fetches 16 tokens of staging row lane / 4, piece lane % 4
        const int rr = lane >> 2, rj = lane & 3;
        const uint32_t raddr = G::chunk(64 * wave + 4 * rr + (rj ^ (rr >> 2)));
        const int orow = tile * TILE_ROWS + rr;
        // row-major: 64-byte steps between the halves; token-tile-major ([M / 32][N][32], tok0 a multiple of 32):
        // piece rj of half h lies in tile tok0 / 32 + rj / 2 + 2 h, at byte 16 (rj & 1) of the row
        const bool ot = (OT == 1) || (OT == -1 && a.out_tile_stride != 0);
        const uint32_t ots = (uint32_t)a.out_tile_stride;
        const uint32_t off = ot ? (uint32_t)((tok0 >> 5) + (rj >> 1)) * ots + (uint32_t)orow * 32u + (uint32_t)((rj & 1) * 16)
                                : (uint32_t)orow * (uint32_t)a.ldo + (uint32_t)(tok0 + 16 * rj);
        const uint32_t half_step = ot ? 2u * ots : 64u;
        const __amdgpu_buffer_rsrc_t rs = out_resource(a);
        // (Sum: read in the accumulator layout, row 16 * tile + c; rows past N are never stored)
        const bool sum_row_ok = tile * TILE_ROWS + c < a.N;
        const float* sp = a.sum + ((uint32_t)(tile * TILE_ROWS + c) * (uint32_t)a.ld_sum + (uint32_t)(tok0 + 4 * g));
#pragma unroll
        for (int h = 0; h < G::HALVES; ++h) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int i = 4 * h + j;
                if (i >= G::PIECES) continue;   // (a 96-token tile ends after piece 5)
                float y[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) y[r] = __fmaf_rn((float)acc[i][r], scale, bias);
                if constexpr ((POST & POST_SUM_BIT) != 0) {
                    if (sum_row_ok && (!CUT || tok0 + 16 * i + 4 * g < a.M)) {
                        v4f t;
                        if constexpr (CUT) t = load_sum4<POST, true>(a, tile * TILE_ROWS + c, tok0 + 16 * i + 4 * g);
                        else t = ((const v4f_any*)(sp + 16 * i))->v;
#pragma unroll
                        for (int r = 0; r < 4; ++r) y[r] = y[r] + t[r];
                    }
                }
                *(uint32_t*)(lds + wbase + (uint32_t)(j ^ wsw) * G::STRIDE) = quantise4<OUT, POST>(a, y, lut);
            }
            const v4i v = *(const v4i*)(lds + raddr);   // same wave: LDS operations complete in order
            const int left = CUT ? a.M - (tok0 + 16 * (4 * h + rj)) : 16;
            if (orow < a.N && 4 * h + rj < G::PIECES && left > 0) {
                if (CUT && left < 16) {
                    store_cut16((uint8_t*)a.out + (off + half_step * h), v, left);
                } else if constexpr (OT == 1) {
                    store16_out<SCOPE_AGENT>(rs, off, v, half_step * h);
                } else if constexpr (OT == 0) {
                    ((v4i_any*)((uint8_t*)a.out + off + half_step * h))->v = v;
                } else {
                    if (ot) store16_out<SCOPE_AGENT>(rs, off, v, half_step * h);
                    else store16_out<SCOPE_DEFAULT>(rs, off, v, half_step * h);
                }
            }
        }
    }
}

// The same for a tile that takes the general path: cut by the end of the tokens, or an output that takes_fast_stores
// refuses.  TIGHT: nothing of it is to stay in registers across the phases (see pinned).
template <int TM, int OUT, int POST, bool WIDE, bool TIGHT, int OT = -1>
__device__ __forceinline__ void finish_tile_any(const Args& a, const v4i (&acc)[Geo<TM>::PIECES], const float scale,
                                                const float bias, const int tile, const int tok0, int lane, const uint8_t* lds)
{
    if constexpr (TIGHT) lane = pinned(lane);
    const int g = lane >> 4, n = tile * TILE_ROWS + (lane & 15);
    if (n < a.N) {
        const LdsLut<TM, TIGHT> lut{lds};
#pragma unroll
        for (int i = 0; i < Geo<TM>::PIECES; ++i) {
            const int m0 = tok0 + 16 * i + 4 * g;
            if (m0 < a.M) finish4<OUT, POST, WIDE, OT>(a, acc[i], scale, bias, n, m0, lut, load_sum4<POST, TIGHT>(a, n, m0));
        }
    }
}

template <int TM, int NW, int MAXS, int OUT, int POST, int LAYOUT = 0>
__global__ void __launch_bounds__(NW * 64) spmm_rowtile_mfma(const KernelArgs args)
{
    const Args a = unpack<OUT>(args);
    using G = Geo<TM>;
    // LAYOUT bit 0: activations token-tile-major; bit 1: (1-byte) outputs token-tile-major
    constexpr int XT = LAYOUT & 1, OTILED = (LAYOUT >> 1) & 1;
    constexpr int NTHREADS = NW * 64;
    constexpr int PIECES = G::PIECES;
    // activation rows one load pass covers: a power of two; with 6 pieces per row only
    // ROWS_PER_PASS * 6 threads (whole waves) stage
    constexpr int ROWS_PER_PASS = (NTHREADS / PIECES >= 128) ? 128 : 64;
    constexpr int STAGERS = ROWS_PER_PASS * PIECES;
    constexpr int XLOADS = SEGMENT_ROWS / ROWS_PER_PASS;            // 16-byte loads per staging thread and phase
    static_assert(STAGERS <= NTHREADS && STAGERS % 64 == 0, "staging threads must be whole waves of the workgroup");
    __shared__ __attribute__((aligned(16))) uint8_t lds[G::LDS];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15;
    // 16 waves have 128 registers each: the thread id is all of a thread's position that is kept across the phases
    constexpr bool TIGHT = NW > 8;
    auto mine = [&]() __attribute__((always_inline)) {
        if constexpr (TIGHT) return pinned(tid);
        else return tid;
    };

    // workgroup -> (row group, token-tile stream)
    const int S = a.n_streams;
    int stream, rg;
    if (!decode_workgroup(a, (a.ntiles + NW - 1) / NW, S, rg, stream)) return;
    const int n_my = a.tiles_per_stream + (stream < (a.M + TM - 1) / TM - a.tiles_per_stream * S ? 1 : 0);   // token tiles of this stream (>= 1)
    const int total = n_my * a.nseg;                                          // phases

    const int tile = rg * NW + wave;
    const bool have_tile = tile < a.ntiles;
    const int n = tile * TILE_ROWS + c;                       // this lane's output row
    // per-lane constants of the post-operators: loaded in the start-up sequence below, behind
    // the activation and weight loads whose latency they would otherwise precede
    int init = 0;
    float scale = 0.0f, bias = 0.0f;

    v4i A0[MAXS], A1[MAXS];
    uint32_t I0[MAXS], I1[MAXS];
    int n0 = 0, n1 = 0;
    constexpr int XH = XLOADS / 2;   // the prefetch is issued and committed in two halves
    static_assert(XH * 2 == XLOADS, "even number of prefetch loads");
    v4i xr[XH];
    v4i acc[PIECES];

    // per-thread staging coordinates: XLOADS rows (ROWS_PER_PASS apart), one 16-byte piece
    const bool stager = (STAGERS == NTHREADS) || wave < STAGERS / 64;

    // Where a phase is, in scalar registers and stepped from one phase to the next: worked out from its number, it took a
    // division at every use, on the vector units and by every wave (2048 x 2048 at 75 %, 4096 tokens: 21.4 -> 20.6 us).
    struct Phase { int seg, tok0; };
    auto after = [&](Phase f) __attribute__((always_inline)) {
        if (++f.seg == a.nseg) { f.seg = 0; f.tok0 += S * TM; }
        return f;
    };
    Phase cur = {0, stream * TM}, nxt_phase = after(cur);

    // ---- global loads of half h of the activations of a phase into registers.  The common case
    // (full token tile) is branch-free so that all loads are in flight
    // together; rows past the end of K are redirected to the last valid row (never multiplied).
    // Two halves (first issued at the start of the previous phase, second half-way through its
    // multiply) keep only XH prefetch registers live.
    auto x_issue_to = [&](v4i (&xr)[XH], const Phase f, const int h) __attribute__((always_inline)) {
        const int tok0 = f.tok0, k0 = f.seg * SEGMENT_ROWS;
        const int last = min(SEGMENT_ROWS, a.K - k0) - 1;
        if (!stager) return;
        const int t = mine(), x_row0 = t / PIECES, x_piece = t % PIECES;
        if constexpr (XT == 0) {
            if (tok0 + TM <= a.M) {
                // 32-bit offsets from a uniform base (x_fast)
                const uint8_t* src = a.X + (int64_t)k0 * a.ldx + tok0;
#pragma unroll
                for (int u = 0; u < XH; ++u) {
                    const int row = min(x_row0 + (h * XH + u) * ROWS_PER_PASS, last);
                    xr[u] = load16_any(src + ((uint32_t)row * (uint32_t)a.ldx + (uint32_t)(x_piece * 16)));
                }
            } else {
                // last, ragged token tile: still one branch-free load per piece
                const RaggedPieces<0> tail(a, k0, last);
                const int col = tok0 + x_piece * 16;
#pragma unroll
                for (int u = 0; u < XH; ++u) xr[u] = tail.load(min(x_row0 + (h * XH + u) * ROWS_PER_PASS, last), col);
                if (!tail.inside) {
#pragma unroll
                    for (int u = 0; u < XH; ++u)
                        xr[u] = tail.shifted(xr[u], min(x_row0 + (h * XH + u) * ROWS_PER_PASS, last), col);
                }
            }
        } else {
            // token-tile-major activations: the layout is 16-byte aligned and padded to whole 32-token tiles, so
            // a piece that starts before M is read whole and one that starts at or after M is not needed at
            // all (its columns are never stored): one branch-free form, no masks, no unaligned path
            const int col = tok0 + x_piece * 16;
            const uint8_t* src = a.X + (int64_t)k0 * 32;
            const uint32_t off = col < a.M ? (uint32_t)xcol<1>(a, col) : 0u;
#pragma unroll
            for (int u = 0; u < XH; ++u) {
                const int row = min(x_row0 + (h * XH + u) * ROWS_PER_PASS, last);
                xr[u] = *(const v4i*)(src + ((uint32_t)row * 32u + off));
            }
        }
    };

    // ---- ... and from registers into LDS buffer q % 2, as x - 128
    auto x_commit_from = [&](const v4i (&xr)[XH], const int q, const int h) {
        if (!stager) return;
        const int t = mine();
        uint8_t* buf = lds + (G::X0 + (q & 1) * G::BUF + h * XH * ROWS_PER_PASS * G::STRIDE) + (t / PIECES * G::STRIDE + t % PIECES * 16);
#pragma unroll
        for (int u = 0; u < XH; ++u)
            *(v4i*)(buf + u * ROWS_PER_PASS * G::STRIDE) = xr[u] ^ (v4i){FLIP, FLIP, FLIP, FLIP};
    };
    auto x_issue = [&](const int h) { x_issue_to(xr, nxt_phase, h); };
    auto x_commit = [&](const int q, const int h) { x_commit_from(xr, q, h); };
    // ---- compressed weights + activation-row indices of (tile, segment of phase q).  Loads are
    // unconditional (slots past the segment's step count re-read step 0 and are never used).
    auto w_issue_at = [&](const int s0, v4i (&A)[MAXS], uint32_t (&I)[MAXS], const int cnt) {
        const int lane = mine() & 63;
#pragma unroll
        for (int s = 0; s < MAXS; ++s) {
            const int step = (s < cnt) ? s0 + s : 0;
            load_step(a, step, lane, A[s], I[s]);
        }
    };
    auto w_issue = [&](const int seg, v4i (&A)[MAXS], uint32_t (&I)[MAXS], int& cnt) {
        cnt = 0;
        int s0 = 0;
        if (have_tile) {
            s0 = a.bounds[tile * (a.nseg + 1) + seg];
            cnt = a.bounds[tile * (a.nseg + 1) + seg + 1] - s0;
        }
        w_issue_at(s0, A, I, cnt);
    };
    // ---- multiply phase q: gather + transpose out of LDS, PIECES matrix instructions per step.
    // Half-way (after step slot MAXS/2 - 1, executed or not) the first half of the next phase's
    // activations is committed and the second half's loads are issued.
    auto multiply = [&](const int q, const bool nxt, const v4i (&A)[MAXS], const uint32_t (&I)[MAXS], const int cnt) {
        const uint32_t base = G::X0 + (uint32_t)(q & 1) * G::BUF + (uint32_t)(mine() & 1) * 8;
#pragma unroll
        for (int s = 0; s < MAXS; ++s) {
            if (s < cnt) {
                // this lane supplies the address of list slot 16g + c/2 (and + 8), token half c & 1
                const uint32_t a0 = first_row(I[s]) * G::STRIDE + base;
                const uint32_t a1 = second_row(I[s]) * G::STRIDE + base;
#pragma unroll
                for (int i = 0; i < PIECES; ++i) {
                    const v2i x0 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i_ptr)(lds + a0 + 16 * i));
                    const v2i x1 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i_ptr)(lds + a1 + 16 * i));
                    const v4i xa = {x0[0], x0[1], x1[0], x1[1]};
                    acc[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xa, A[s], acc[i], 0, 0, 0);
                }
            }
            if (s == MAXS / 2 - 1 && nxt) {
                x_commit(q + 1, 0);
                x_issue(1);
            }
        }
    };
    // ---- after the last segment of a token tile: post-operators, store, reset accumulators
    // (16 waves with 6 step slots spill with a second copy of the staged stores)
    constexpr bool CUT_FAST = (OUT == SPMM_OUT_S8 || OUT == SPMM_OUT_U8) && !(NW == 16 && MAXS == 6);
    auto finish = [&]() __attribute__((always_inline)) {
        if (cur.seg != a.nseg - 1) return;
        const bool fast_out = takes_fast_stores<OUT>(a);
        const int tok0 = cur.tok0;
        const int lane = mine() & 63;
        if (have_tile) {
            if (fast_out && tok0 + TM <= a.M) {
                finish_tile_fast<TM, OUT, POST, OTILED, NW == 16 && MAXS == 6>(a, acc, scale, bias, tile, tok0, lane, wave, lds);
            } else if (CUT_FAST && fast_out) {
                finish_tile_fast<TM, OUT, POST, OTILED, false, true>(a, acc, scale, bias, tile, tok0, lane, wave, lds);
            } else {
                finish_tile_any<TM, OUT, POST, NW != 16, TIGHT, OTILED>(a, acc, scale, bias, tile, tok0, lane, lds);
            }
        }
#pragma unroll
        for (int i = 0; i < PIECES; ++i) acc[i] = (v4i){init, init, init, init};
    };
    const bool reload = a.nseg > 2;   // otherwise set q % 2 always holds segment q % nseg

    {   // ---- start-up: every load of the first phase is issued before anything waits -- both
        // halves of the activations (the second in registers that are not live yet), the weights,
        // then the per-lane constants and the table -- and consumed in that order
        v4i x2[XH];
        // (the step range of the first weights: a scalar load whose latency the address arithmetic
        // of the activation loads covers)
        int w_s0 = 0;
        if (have_tile) {
            w_s0 = a.bounds[tile * (a.nseg + 1)];
            n0 = a.bounds[tile * (a.nseg + 1) + 1] - w_s0;
        }
        x_issue_to(xr, cur, 0);
        x_issue_to(x2, cur, 1);
        w_issue_at(w_s0, A0, I0, n0);
        if (have_tile) init = a.rowsum[n] * a.corr_mul;
        if constexpr (OUT != SPMM_OUT_S32) {
            if (have_tile && n < a.N) {
                scale = a.w_scale[n] * a.x_scale;
                if (a.bias) bias = a.bias[n];
            }
        }
        constexpr bool TABLE = (POST & SPMM_POST_GELU) != 0 && (OUT == SPMM_OUT_S8 || OUT == SPMM_OUT_U8);
        int table_byte = 0;
        if constexpr (TABLE) {
            if (tid < 256) table_byte = a.lut[tid];
        }
        x_commit_from(xr, 0, 0);
        x_commit_from(x2, 0, 1);
        if constexpr (TABLE) {
            if (tid < 256) lds[G::lut_addr(tid)] = (uint8_t)table_byte;
        }
    }
#pragma unroll
    for (int i = 0; i < PIECES; ++i) acc[i] = (v4i){init, init, init, init};
    wait_global_loads();
    __syncthreads();
    for (int p = 0; p < total; p += 2) {
        {   // even phase: register set 0, LDS buffer 0
            const bool nxt = p + 1 < total;
            if (nxt) {
                x_issue(0);
                if (reload || p + 1 < 2) w_issue(nxt_phase.seg, A1, I1, n1);
            }
            multiply(p, nxt, A0, I0, n0);
            if (nxt) x_commit(p + 1, 1);
            wait_global_loads();   // before the output stores: they must not be waited for
            finish();
            cur = nxt_phase;
            nxt_phase = after(cur);
            __syncthreads();
        }
        if (p + 1 >= total) break;
        {   // odd phase: register set 1, LDS buffer 1
            const bool nxt = p + 2 < total;
            if (nxt) {
                x_issue(0);
                if (reload) w_issue(nxt_phase.seg, A0, I0, n0);
            }
            multiply(p + 1, nxt, A1, I1, n1);
            if (nxt) x_commit(p + 2, 1);
            wait_global_loads();
            finish();
            cur = nxt_phase;
            nxt_phase = after(cur);
            __syncthreads();
        }
    }
}

// =======================================================================================
// Pipelined persistent kernel with loader waves: the same decomposition, LDS geometry and
// phases as spmm_rowtile_mfma, but the workgroup is NW compute waves (one row tile each)
// plus LW = 4 waves that do nothing but stage the activations.
//
// Why: on this architecture loads and stores of a wave share one completion counter and may
// complete out of order with each other, so a wave that has stored a tile's outputs cannot
// wait for its next activation loads without also waiting until the stores have reached
// memory.  In spmm_rowtile_mfma every wave does both, and for 4-byte outputs (the downconvert
// of Section 3.3 left out: 4 N M bytes) the whole workgroup then stands still at the next
// commit until the burst of stores has drained.  Here the waves that store never load
// activations (with at most two K segments they load nothing at all after start-up), and the
// waves that load never store: the stores of tile j drain while tile j + 1 is multiplied.
//
// Loader wave: at the start of phase p its registers hold the activations of phase p + 1
// (requested a whole phase earlier); it writes them to buffer (p + 1) % 2, whose readers
// finished before the last barrier, requests phase p + 2 and goes to the barrier.
// Compute wave: multiply out of buffer p % 2, post-operators after the last segment, barrier.
// Both kinds pass exactly 1 + phases barriers.
// =======================================================================================
template <int TM, int NW, int LW, int MAXS, int OUT, int POST>
__global__ void __launch_bounds__((NW + LW) * 64) spmm_rowtile_mfma_fed(const KernelArgs args)
{
    const Args a = unpack<OUT>(args);
    using G = Geo<TM>;
    constexpr int PIECES = G::PIECES;
    constexpr int LTHREADS = LW * 64;
    constexpr int ROWS_PER_PASS = TM == 64 ? 64 : 32;
    constexpr int STAGERS = ROWS_PER_PASS * PIECES;              // 256 (128 or 64 tokens) or 192 (96 tokens)
    constexpr int XLOADS = SEGMENT_ROWS / ROWS_PER_PASS;         // 16-byte loads per staging thread and phase
    static_assert(STAGERS <= LTHREADS, "the loader waves must cover one pass of rows");
    __shared__ __attribute__((aligned(16))) uint8_t lds[G::LDS];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, c = lane & 15;
    // the forms whose weights and accumulators take most of the 128 registers that each of 16 waves has (see pinned)
    constexpr bool FULL = NW > 8 && MAXS > 4 && TM > 64;

    // workgroup -> (row group, token-tile stream)
    const int S = a.n_streams;
    int stream, rg;
    if (!decode_workgroup(a, (a.ntiles + NW - 1) / NW, S, rg, stream)) return;
    const int n_my = a.tiles_per_stream + (stream < (a.M + TM - 1) / TM - a.tiles_per_stream * S ? 1 : 0);
    const int total = n_my * a.nseg;                                          // phases
    // where a phase is (see spmm_rowtile_mfma)
    struct Phase { int seg, tok0; };
    auto after = [&](Phase f) __attribute__((always_inline)) {
        if (++f.seg == a.nseg) { f.seg = 0; f.tok0 += S * TM; }
        return f;
    };
    Phase cur = {0, stream * TM};
    constexpr bool TABLE = (POST & SPMM_POST_GELU) != 0 && (OUT == SPMM_OUT_S8 || OUT == SPMM_OUT_U8);

    if (wave >= NW) {
        // ------------------------------------------------------------------ loader wave
        const int ltid = tid - NW * 64;
        const bool stager = ltid < STAGERS;
        const int x_row0 = ltid / PIECES, x_piece = ltid % PIECES;
        const uint32_t x_lds0 = G::X0 + (uint32_t)x_row0 * G::STRIDE + x_piece * 16;
        const uint32_t x_off = (uint32_t)xcol(a, x_piece * 16);
        v4i xr[XLOADS];
        auto x_issue = [&]() __attribute__((always_inline)) {   // (and steps to the next phase)
            const int tok0 = cur.tok0, k0 = cur.seg * SEGMENT_ROWS;
            cur = after(cur);
            const int last = min(SEGMENT_ROWS, a.K - k0) - 1;   // rows past K repeat the last one (never multiplied)
            if (!stager) return;
            if (tok0 + TM <= a.M) {
                const uint8_t* src = a.X + (int64_t)k0 * a.ldx + xcol(a, tok0);
                const uint32_t ldx = (uint32_t)a.ldx;
                const uint32_t first = (uint32_t)x_row0 * ldx + x_off, end = (uint32_t)last * ldx + x_off;
#pragma unroll
                for (int u = 0; u < XLOADS; ++u)
                    xr[u] = load16_any(src + min(first + (uint32_t)(u * ROWS_PER_PASS) * ldx, end));
            } else {
                // last, ragged token tile: still one branch-free load per piece
                const RaggedPieces<> tail(a, k0, last);
                const int col = tok0 + x_piece * 16;
#pragma unroll
                for (int u = 0; u < XLOADS; ++u) xr[u] = tail.load(min(x_row0 + u * ROWS_PER_PASS, last), col);
                if (!tail.inside) {
#pragma unroll
                    for (int u = 0; u < XLOADS; ++u)
                        xr[u] = tail.shifted(xr[u], min(x_row0 + u * ROWS_PER_PASS, last), col);
                }
            }
        };
        auto x_commit = [&](const int q) {
            if (!stager) return;
            uint8_t* buf = lds + (q & 1) * G::BUF + x_lds0;
#pragma unroll
            for (int u = 0; u < XLOADS; ++u)
                *(v4i*)(buf + u * ROWS_PER_PASS * G::STRIDE) = xr[u] ^ (v4i){FLIP, FLIP, FLIP, FLIP};
        };
        x_issue();
        int table_byte = 0;
        if constexpr (TABLE) table_byte = a.lut[ltid];          // LTHREADS == 256 entries
        x_commit(0);
        if constexpr (TABLE) lds[G::lut_addr(ltid)] = (uint8_t)table_byte;
        if (1 < total) x_issue();
        __syncthreads();
        for (int p = 0; p < total; ++p) {
            if (p + 1 < total) x_commit(p + 1);
            if (p + 2 < total) x_issue();
            __syncthreads();
        }
        return;
    }

    // ---------------------------------------------------------------------- compute wave
    const int tile = rg * NW + wave;
    const bool have_tile = tile < a.ntiles;
    const int n = tile * TILE_ROWS + c;                       // this lane's output row
    int init = 0;
    float scale = 0.0f, bias = 0.0f;
    v4i A0[MAXS], A1[MAXS];
    uint32_t I0[MAXS], I1[MAXS];
    v4i acc[PIECES];

    // Steps of (tile, segment of phase q).  Read a phase before they are needed: a scalar load whose latency would
    // otherwise precede every phase's weights.
    struct Range { int first, count; };
    int w_seg = 0;                                            // of the next phase whose range will be read
    auto next_range = [&](const int q) {                      // (phase q's)
        Range r = {0, 0};
        if (have_tile && q < total) {
            const int32_t* const b = a.bounds + (int64_t)tile * (a.nseg + 1) + w_seg;
            r.first = b[0];
            r.count = b[1] - r.first;
        }
        if (++w_seg == a.nseg) w_seg = 0;
        return r;
    };
    auto w_issue = [&](const Range r, v4i (&A)[MAXS], uint32_t (&I)[MAXS]) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < MAXS; ++s)
            if (s < r.count) load_step(a, r.first + s, lane, A[s], I[s]);
    };
    // Multiply phase q.  With LOAD the weights of the next phase are requested on the way, two step slots at a time:
    // issued in one go they kept the wave from its first gather for as long as the CU's address path took to
    // work through everyone's requests (4096 x 4096 at 85 %, 1024 tokens, cycles per phase: 1000-1350 issuing, then
    // 1800-2150 multiplying).  They have landed when the phase ends, and are waited for there, before any store.
    auto multiply = [&](auto LOAD, const int q, const v4i (&A)[MAXS], uint32_t (&I)[MAXS], const int cnt,
                        v4i (&An)[MAXS], uint32_t (&In)[MAXS], const Range next) __attribute__((always_inline)) {
        const uint32_t base = G::X0 + (uint32_t)(q & 1) * G::BUF + (c & 1) * 8;
#pragma unroll
        for (int s = 0; s < MAXS; ++s) {
            if constexpr (LOAD.value) {
#pragma unroll
                for (int l = 2 * s; l < min(2 * s + 2, MAXS); ++l)
                    if (l < next.count) load_step(a, next.first + l, lane, An[l], In[l]);
            }
            if (s < cnt) {
                // Weights that stay: or their rows' LDS addresses would be kept beside them, two registers for each one.
                // Reloaded ones, 8 slots: or the compiler has int32 outputs wait for everything outstanding, the last
                // tile's stores included, before each request (3072 x 3072 at 70 %, 4096 tokens: 70.1 -> 56.9 us; 2944 x
                // 2944 at 73 %, 1982 tokens 35.8 -> 30.2; other outputs within 0.4 %, or faster by up to 4).
                if constexpr (LOAD.value ? MAXS == 8 : FULL) I[s] = pinned(I[s]);
                const uint32_t a0 = first_row(I[s]) * G::STRIDE + base;
                const uint32_t a1 = second_row(I[s]) * G::STRIDE + base;
#pragma unroll
                for (int i = 0; i < PIECES; ++i) {
                    const v2i x0 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i_ptr)(lds + a0 + 16 * i));
                    const v2i x1 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i_ptr)(lds + a1 + 16 * i));
                    const v4i xa = {x0[0], x0[1], x1[0], x1[1]};
                    acc[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xa, A[s], acc[i], 0, 0, 0);
                }
            }
        }
    };
    // (The forms without registers for a second copy of the staged stores do without: they spill, or, 12 waves with 6 step
    // slots on 96 tokens, are slower for it: 2304x768 at 85 %, 1771 tokens, s8 9.6 and 9.9 us.)
    constexpr bool CUT_FAST = (OUT == SPMM_OUT_S8 || OUT == SPMM_OUT_U8) &&
                              (MAXS == 4 || (NW == 8 && MAXS == 6) || (TM == 64 && !(POST & POST_SUM_BIT)));
    auto finish = [&]() __attribute__((always_inline)) {        // (and steps to the next phase)
        const Phase at = cur;
        cur = after(cur);
        if (at.seg != a.nseg - 1) return;
        const bool fast_out = takes_fast_stores<OUT>(a);
        const int tok0 = at.tok0;
        if (have_tile) {
            if (fast_out && tok0 + TM <= a.M) {
                finish_tile_fast<TM, OUT, POST>(a, acc, scale, bias, tile, tok0, lane, wave, lds);
            } else if (CUT_FAST && fast_out) {
                finish_tile_fast<TM, OUT, POST, -1, false, true>(a, acc, scale, bias, tile, tok0, lane, wave, lds);
            } else if constexpr (FULL && (POST & POST_SUM_BIT) && (OUT == SPMM_OUT_S8 || OUT == SPMM_OUT_U8)) {
                finish_tile_any<TM, OUT, POST, false, FULL>(a, acc, scale, bias, tile, tok0, lane, lds);
            } else if (n < a.N) {
                // (finish_tile_any but for the pin, which costs more than it saves where nothing spills without it: 3018 x 3018
                // at 86 %, 1886 tokens, GELU to binary32: 19.7 us, with it 20.3)
                const LdsLut<TM> lut{lds};
#pragma unroll
                for (int i = 0; i < PIECES; ++i) {
                    const int m0 = tok0 + 16 * i + 4 * g;
                    if (m0 < a.M) finish4<OUT, POST, false>(a, acc[i], scale, bias, n, m0, lut, load_sum4<POST, FULL>(a, n, m0));
                }
            }
        }
#pragma unroll
        for (int i = 0; i < PIECES; ++i) acc[i] = (v4i){init, init, init, init};
    };
    Range r0 = next_range(0), r1 = next_range(1);
    // (the first weights lie where tile_steps says: requested without waiting for the bounds)
    Range early = r0;
    if (a.tile_steps && have_tile) early = {tile * a.tile_steps, a.tile_steps};
    w_issue(early, A0, I0);
    if (have_tile) init = a.rowsum[n] * a.corr_mul;
    if constexpr (OUT != SPMM_OUT_S32) {
        if (have_tile && n < a.N) {
            scale = a.w_scale[n] * a.x_scale;
            if (a.bias) bias = a.bias[n];
        }
    }
#pragma unroll
    for (int i = 0; i < PIECES; ++i) acc[i] = (v4i){init, init, init, init};
    // register set p % 2 holds the weights of phase p: with at most two segments for the whole kernel, otherwise
    // reloaded a phase ahead
    auto phases = [&](auto RELOAD) __attribute__((always_inline)) {
        if constexpr (!RELOAD.value) w_issue(r1, A1, I1);
        __syncthreads();
        for (int p = 0; p < total; p += 2) {
            {   // even phase: register set 0, LDS buffer 0
                const int cnt = r0.count;
                if constexpr (RELOAD.value) r0 = next_range(p + 2);
                multiply(RELOAD, p, A0, I0, cnt, A1, I1, r1);
                if constexpr (RELOAD.value) wait_global_loads();
                finish();
                __syncthreads();
            }
            if (p + 1 >= total) break;
            {   // odd phase: register set 1, LDS buffer 1
                const int cnt = r1.count;
                if constexpr (RELOAD.value) r1 = next_range(p + 3);
                multiply(RELOAD, p + 1, A1, I1, cnt, A0, I0, r0);
                if constexpr (RELOAD.value) wait_global_loads();
                finish();
                __syncthreads();
            }
        }
    };
    if (a.nseg > 2) phases(std::true_type{});
    else phases(std::false_type{});
}

// =======================================================================================
// Short batches: the simple kernel (token tile 64, 32 or 16, any K) and the short-batch kernel with 16-token
// tiles (K <= 4096) are one body with different amounts of resident K.
//
// A launch here is a few microseconds long, and its time is a chain of memory latencies and of the instructions between them:
// a wave issues a vector instruction every 4 cycles, every 8 where two share a SIMD, and a kernel of 2000 cycles has no room for a
// hundred that do nothing for it.  So what a workgroup needs is requested in the order in which it is needed: the whole [K x TM]
// slab of activations, in code without branches for 1, 2, 4 .. passes of rows; the first weights of every wave (whose place
// follows from tile_steps, without reading the bounds), a branch for each set after the first, so that short shares issue
// nothing in vain (without these branches each wait is for what it needs alone, but calls are 5 to 30 % slower); the per-row
// constants, the operand of Sum, the table.  Divisions are shifts, addresses 32-bit offsets; what only K beyond the RES resident
// rows or far rows need is behind one branch (worked out ahead of a loop for both, it took 700 cycles between the barrier and the
// first step).  The slab then goes to LDS, one barrier, and each wave walks its steps in groups of CH, branch-free inside a group
// (steps past the end read as zero weights), the weights of the next NS - 1 groups in flight.  Kernel times against the ones
// before, which had a branch per pass and step, divisions and a wait for everything (profiles/spmm_resident_kernel_times.txt, 360
// problems), us: 256x256 at 90 %, 128 tokens 3.8 -> 2.8; 3072x768 at 85 %, 128 tokens, u8 with GELU 4.8 -> 3.9; 768x3072 at 80 %,
// 333 tokens with Sum, binary32 10.3 -> 9.3; 2944x2944 at 80 %, 16 tokens 5.1 -> 3.9; calls of less than 4 us are bound by the
// host's launches.
//
// LDS: a row is TM bytes, unpadded.  Two workgroups share a CU (one of the slab, and one with pairs of row tiles, R = 2, which have
// more than 128 registers); with 16-token tiles four would have the LDS, with 32 and 64 tokens two.  A row's 16-byte pieces are
// rotated by an xor with bits of the row number such that rows whose numbers differ mod 16 (the packer's order) lie in 16 different
// groups of four banks.
//
// A workgroup has 8 waves and 8, 4 or 2 row tiles (Args::wg_tiles): with fewer than 8, the waves share the row
// tiles, each taking a part of its steps, and the partial sums meet in LDS.  For grids that leave most of the
// chip idle: fewer rows per workgroup, more CUs.
// =======================================================================================
template <int TM>
struct Swizzle {
    // byte offset of 16-byte piece 0 of activation row r; piece i is at offset ^ 16 i
    static __device__ __forceinline__ uint32_t row(const uint32_t r)
    {
        if constexpr (TM == 16) return r * 16;
        else if constexpr (TM == 32) return r * 32 + (r << 1 & 16);
        else return r * 64 + (r << 2 & 48);
    }
};

template <int TM, int R, int RES, int OUT, int POST>
struct Resident {
    static_assert(TM == 64 || TM == 32 || TM == 16, "token tile of the short-batch kernels");
    static constexpr int PIECES = TM / 16, THREADS = 512;
    static constexpr int PASS_ROWS = THREADS / PIECES;          // activation rows one load pass covers
    static constexpr int PASSES = RES / PASS_ROWS;
    static constexpr int SEGS = RES / SEGMENT_ROWS;             // segments per round
    // weights in flight: NS sets of CH steps, gathered CH steps at a time (the slabs have 256 registers, the others
    // 128, for two workgroups on a CU; with R = 2 up to 147, and one)
    static constexpr bool WIDE = RES > 2048;
    static constexpr int CH = TM == 16 || WIDE ? 4 : 2;
    static constexpr int NS = TM == 16 ? (WIDE ? 6 : 3) : WIDE ? 5 : TM == 32 ? 4 : 3;
    // LDS: activations, the table, and what the waves that share a row tile hand to the first of them: of 6 waves at most
    // (64-token workgroups have 8 row tiles, or pairs)
    static constexpr bool SHARES = R == 1 && TM < 64;
    static constexpr int TABLE_AT = RES * TM, SUMS_AT = TABLE_AT + 256, LDS = SUMS_AT + (SHARES ? 6 * PIECES * 1024 : 0);
    // The operand of Sum is requested with everything else at the start, where the grid is one round of workgroups, as
    // it is with narrow tiles: its latency is hidden (768 x 768, 128 tokens: 4.76 us, requested after the last step 4.90).
    // 64-token tiles are planned for grids of several rounds, where the second workgroup on a CU is worth more than that
    // and the 16 registers of the operand would cost it (145 of 128): 2688 x 672 at 71 %, 1400 tokens, binary32: 15.8 ->
    // 11.6 us, 2800 tokens 28.7 -> 20.0, int8 26.3 -> 19.0; 800 x 800 at 72 %, 5024 tokens 19.3 -> 17.2.
    static constexpr bool SUM = (POST & POST_SUM_BIT) != 0, SUM_LATE = TM == 64;
    static constexpr bool TABLE = (POST & SPMM_POST_GELU) != 0 && (OUT == SPMM_OUT_S8 || OUT == SPMM_OUT_U8);
    static_assert((RES & (RES - 1)) == 0 && PASSES * PASS_ROWS == RES && SEGMENT_ROWS % PASS_ROWS == 0, "threads tile a segment");

    static __device__ __forceinline__ uint32_t row_offset(const uint32_t r) { return Swizzle<TM>::row(r); }

    static __device__ __forceinline__ void run(const Args& a, uint8_t* const lds)
    {
        // (row tiles per workgroup and waves per row tile are powers of two: everything here is a shift)
        const int wt = __builtin_ctz((unsigned)a.wg_tiles), kb = 3 - wt;
        const int group_bits = wt + (R == 2 ? 1 : 0);
        int tt, rg;
        if (!decode_tile(a, (a.ntiles + (1 << group_bits) - 1) >> group_bits, (a.M + TM - 1) / TM, rg, tt)) return;
        const int tid = threadIdx.x;
        const int lane = tid & 63;
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int g = lane >> 4, c = lane & 15;
        const int tok0 = tt * TM;
        const int part = wave & ((1 << kb) - 1), local = wave >> kb;      // 1, 2 or 4 waves share a row tile
        const int tile0 = ((rg << wt) + local) * R;             // this wave's first row tile
        const bool have = tile0 < a.ntiles;

        // ---- weights: NS rotating sets of CH steps of this wave's share of a row tile's steps.  The resource ends with the share:
        // a load past it gives zeros, and fetches nothing.
        v4i A[NS][CH];
        uint32_t I[NS][CH];
        __amdgpu_buffer_rsrc_t share;
        int from = 0, steps = 0;                                // of the share
        const int val_at = lane * 16, row_at = STEP_VAL_BYTES + 32 * g + 4 * (c >> 1);
        // The same in every lane, and said so: with bounds from vector loads the compiler otherwise loops over the lanes around each
        // weight load (kernels with a table: 195 such loops with 16-token tiles, 22 KB of code instead of 11; u8 with GELU,
        // 3072x768 at 85 %, 128 tokens 4.1 us instead of 3.9; s8, 768x4096 at 80 %, 333 tokens 12.4 instead of 10.6).
        auto w_open = [&](const int first_, const int all_) __attribute__((always_inline)) {      // steps first .. first + all - 1 of the weight
            const int first = __builtin_amdgcn_readfirstlane(first_), all = __builtin_amdgcn_readfirstlane(all_);
            from = first + (all * part >> kb);
            steps = first + (all * (part + 1) >> kb) - from;
            share = __builtin_amdgcn_make_buffer_rsrc((void*)(a.records + (int64_t)from * RECORD_BYTES), 0, steps * RECORD_BYTES, 0x00020000);
        };
        auto w_load = [&](v4i (&w)[CH], uint32_t (&rows)[CH], const int step) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < CH; ++j) rows[j] = __builtin_amdgcn_raw_buffer_load_b32(share, row_at + j * RECORD_BYTES, step * RECORD_BYTES, 0);
#pragma unroll
            for (int j = 0; j < CH; ++j)
                w[j] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(share, val_at + j * RECORD_BYTES, step * RECORD_BYTES, 0));
        };
        auto w_first = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < NS; ++k)
                if (k == 0 || k * CH < steps) w_load(A[k], I[k], k * CH);
        };

        v4i acc[R][PIECES];
        int rowsum[R];
        float scale[R], bias[R];
        v4f sum4[R][PIECES];
        int table_byte = 0;
        // ---- per-row constants, table, operand of Sum: requested, used when the last step has been multiplied
        auto constants = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int n = (tile0 + r) * TILE_ROWS + c, nn = min(n, a.N - 1);      // (rows past the last one are not stored)
                rowsum[r] = a.rowsum[nn];
                scale[r] = bias[r] = 0.0f;
                if constexpr (OUT != SPMM_OUT_S32) {
                    scale[r] = a.w_scale[nn];
                    if (a.bias) bias[r] = a.bias[nn];
                }
#pragma unroll
                for (int i = 0; i < PIECES; ++i) {
                    acc[r][i] = (v4i){0, 0, 0, 0};
                    sum4[r][i] = (v4f){0.0f, 0.0f, 0.0f, 0.0f};
                    const int m0 = tok0 + 16 * i + 4 * g;
                    if (SUM && !SUM_LATE && part == 0 && n < a.N && m0 < a.M) sum4[r][i] = load_sum4<POST>(a, n, m0);
                }
            }
            if (TABLE && tid < 256) table_byte = a.lut[tid];
        };

        // ---- activations: 16-byte pieces, written to LDS as x - 128
        const int x_row = tid / PIECES, x_col = tok0 + tid % PIECES * 16;
        const uint32_t x_lds = row_offset((uint32_t)x_row) ^ (uint32_t)(tid % PIECES * 16);
        const bool cut = tok0 + TM > a.M && a.x_tile_stride == 0;      // (tile-major rows are padded)
        constexpr v4i FLIPS = {FLIP, FLIP, FLIP, FLIP};

        // ---- multiply the share of row tile r
        auto multiply = [&](const int r) __attribute__((always_inline)) {
            for (int s = 0; s < steps; s += NS * CH) {
#pragma unroll
                for (int k = 0; k < NS; ++k) {
                    const int at = s + k * CH;
                    if (at < steps) {
                        v2i x[CH][PIECES][2];
#pragma unroll
                        for (int j = 0; j < CH; ++j) {
                            constexpr uint32_t mask = RES - 1;
                            const uint32_t o0 = row_offset(I[k][j] & mask) + (c & 1) * 8;
                            const uint32_t o1 = row_offset(I[k][j] >> 16 & mask) + (c & 1) * 8;
#pragma unroll
                            for (int i = 0; i < PIECES; ++i) {
                                x[j][i][0] = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i_ptr)(lds + (o0 ^ 16 * i)));
                                x[j][i][1] = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i_ptr)(lds + (o1 ^ 16 * i)));
                            }
                        }
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int j = 0; j < CH; ++j) {
#pragma unroll
                            for (int i = 0; i < PIECES; ++i) {
                                const v4i xa = {x[j][i][0][0], x[j][i][0][1], x[j][i][1][0], x[j][i][1][1]};
                                acc[r][i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xa, A[k][j], acc[r][i], 0, 0, 0);
                            }
                        }
                        if (at + NS * CH < steps) w_load(A[k], I[k], at + NS * CH);
                    }
                }
            }
        };
        // row tile r, segments seg0 .. seg0 + SEGS - 1 (placed: all of it, where tile_steps says; its records past its own steps are zero)
        auto begin = [&](const int r, const int seg0, const bool placed = false) __attribute__((always_inline)) {
            int first = (tile0 + r) * a.tile_steps, count = a.tile_steps;
            if (!placed) {
                const int32_t* const b = a.bounds + (int64_t)min(tile0 + r, a.ntiles - 1) * (a.nseg + 1);
                first = b[seg0];
                count = b[min(seg0 + SEGS, a.nseg)] - first;
            }
            w_open(first, have ? count : 0);
            w_first();
        };

        // All of K resident, and 32-bit offsets: no wait from the first request to the first piece written, and no branch on the way
        // to it, for 1, 2, 4 .. passes of rows.
        auto all_at_once = [&](auto PASSES_) __attribute__((always_inline)) {
            constexpr int P = PASSES_.value;
            v4i xs[P];
            // (rows past K, never multiplied, read what lies there, or the matrix's last bytes)
            const uint32_t x_at = (uint32_t)x_row * (uint32_t)a.ldx + (uint32_t)xcol(a, TM == 16 || x_col < a.M ? x_col : 0);
#pragma unroll
            for (int u = 0; u < P; ++u)
                xs[u] = load16_any(a.X + min(x_at + (uint32_t)(u * PASS_ROWS) * (uint32_t)a.ldx, (uint32_t)a.x_last16));
            const int end = a.bounds[(int64_t)min(tile0, a.ntiles - 1) * (a.nseg + 1) + a.nseg];
            begin(0, 0, a.tile_steps != 0);
            constants();
            auto store = [&]() __attribute__((always_inline)) {
#pragma unroll
                for (int u = 0; u < P; ++u) *(v4i*)(lds + x_lds + u * PASS_ROWS * TM) = xs[u] ^ FLIPS;
            };
            if (__builtin_expect(cut, 0)) {
                const RaggedPieces<> last(a, 0, a.K - 1);      // (all of it as one segment; the last rows' pieces are shifted)
                if (!last.inside) {
#pragma unroll
                    for (int u = 0; u < P; ++u) xs[u] = last.shifted(xs[u], min(x_row + u * PASS_ROWS, a.K - 1), x_col);
                }
                store();
            } else {
                store();
            }
            if (TABLE && tid < 256) lds[TABLE_AT + tid] = (uint8_t)table_byte;
            __syncthreads();
            // A placed tile's steps were requested up to the longest tile's number; those that it does not have (up to half as many
            // again, pack.cpp) are not walked.  One tile in eight 1.4 times as long as the mean: 1024x1024 at 72 %, 2048 tokens,
            // 32-token tiles 8.7 -> 7.8 us; 2048x3072, 1024 tokens, slab 34.6 -> 31.8; even weights 0.95 to 1.01 of the time.
            steps = min(steps, end - from);
            multiply(0);
            if (R == 2 && tile0 + 1 < a.ntiles) {
                begin(1, 0);
                multiply(1);
            }
        };
        // K round by round, and rows that one 32-bit offset does not reach: here too a round's activations and weights are all
        // requested before anything waits (1024x4096 at 80 %, 256 tokens, 64-token tiles: 14.9 us, pass after pass and the
        // weights last 18.8).  Only FAR rows, beyond the offsets of a single pass, or an X of less than 16 bytes, come piece by
        // piece; code of their own keeps the registers of the others within 128.
        auto by_rounds = [&](auto FAR_) __attribute__((always_inline)) {
            constexpr bool FAR = FAR_.value;
            constants();
#pragma unroll 1
            for (int r0 = 0, seg0 = 0; r0 < a.K; r0 += RES, seg0 += SEGS) {
                const int t = pinned_in_turn(tid, r0), row = t / PIECES, col = tok0 + t % PIECES * 16;
                uint8_t* const to = lds + (row_offset((uint32_t)row) ^ (uint32_t)(t % PIECES * 16));
                // (rows past K repeat the last one of their pass, never multiplied)
                v4i xs[PASSES];
                if constexpr (!FAR) {
#pragma unroll
                    for (int u = 0; u < PASSES; ++u) {
                        const int left = a.K - r0 - u * PASS_ROWS;
                        if (left > 0) xs[u] = RaggedPieces<>(a, a.K - left, PASS_ROWS - 1).load(min(row, left - 1), col);
                    }
                }
                begin(0, seg0);
                if (r0 > 0) __syncthreads();   // everyone has finished reading the last round
                if constexpr (!FAR) {
#pragma unroll
                    for (int u = 0; u < PASSES; ++u) {
                        const int left = a.K - r0 - u * PASS_ROWS;
                        if (left > 0) {
                            if (__builtin_expect(cut, 0)) {
                                const RaggedPieces<> pieces(a, a.K - left, min(PASS_ROWS, left) - 1);
                                if (!pieces.inside) xs[u] = pieces.shifted(xs[u], min(row, left - 1), col);
                            }
                            *(v4i*)(to + u * PASS_ROWS * TM) = xs[u] ^ FLIPS;
                        }
                    }
                } else {
#pragma unroll 1
                    for (int k0 = r0; k0 < min(r0 + RES, a.K); k0 += PASS_ROWS)
                        *(v4i*)(to + (k0 - r0) * TM) = load_x16_far(a, min(k0 + row, a.K - 1), col) ^ FLIPS;
                }
                __syncthreads();
                multiply(0);
                if (R == 2 && tile0 + 1 < a.ntiles) {
                    begin(1, seg0);
                    multiply(1);
                }
            }
            // (not before the bounds have been read: they would no longer be scalar loads, in the other path neither)
            if constexpr (TABLE) {
                if (tid < 256) lds[TABLE_AT + tid] = (uint8_t)table_byte;
                __syncthreads();
            }
        };
        // (32-bit offsets: those of X's own rows are below 2^31 + 16, and rows past K, fewer than there are of them or within a pass,
        // do not wrap; RaggedPieces caps its limit there.  768x1024 at 80 %, 100 tokens, a pitch of 1.5 MB, u8 with GELU: 3.77 us,
        // by rounds 4.06; beyond the line, where address translation bounds both, no different.)
        if (__builtin_expect(a.K <= RES && a.x_fast && a.x_last16 < 0x7fffffff, 1)) {
            const int passes = (a.K + PASS_ROWS - 1) / PASS_ROWS;
            if (passes <= 1) all_at_once(std::integral_constant<int, 1>{});
            else if (passes <= 2) all_at_once(std::integral_constant<int, 2>{});
            else if (PASSES == 4 || passes <= 4) all_at_once(std::integral_constant<int, 4>{});
            else all_at_once(std::integral_constant<int, PASSES>{});
        } else if (a.x_fast) {
            by_rounds(std::false_type{});
        } else {
            by_rounds(std::true_type{});
        }

        if (SHARES && kb > 0) {
            v4i* const sums = (v4i*)(lds + SUMS_AT) + (local * ((1 << kb) - 1) - 1) * PIECES * 64 + lane;      // (of part 0; part 1 is the first)
            if (part > 0) {
#pragma unroll
                for (int i = 0; i < PIECES; ++i) sums[(part * PIECES + i) * 64] = acc[0][i];
            }
            __syncthreads();
            if (part > 0) return;
            for (int q = 1; q < 1 << kb; ++q)
#pragma unroll
                for (int i = 0; i < PIECES; ++i) acc[0][i] = acc[0][i] + sums[(q * PIECES + i) * 64];
        }

        const LdsTable lut{lds + TABLE_AT};
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int n = (tile0 + r) * TILE_ROWS + c;
            if (n >= a.N) continue;
            if constexpr (SUM && SUM_LATE) {
#pragma unroll
                for (int i = 0; i < PIECES; ++i) {
                    const int m0 = tok0 + 16 * i + 4 * g;
                    if (m0 < a.M) sum4[r][i] = load_sum4<POST>(a, n, m0);
                }
            }
            const int init = rowsum[r] * a.corr_mul;
#pragma unroll
            for (int i = 0; i < PIECES; ++i) {
                const int m0 = tok0 + 16 * i + 4 * g;
                const v4i sum = acc[r][i] + (v4i){init, init, init, init};
                if (m0 < a.M) finish4<OUT, POST, true>(a, sum, scale[r] * a.x_scale, bias[r], n, m0, lut, sum4[r][i]);
            }
        }
    }
};

// =======================================================================================
// Ring (the streamed kernel: token tile 64, 32 or 16, any K; and the 32-token short-batch kernel): mid-size
// batches, one workgroup of 8 row tiles x TM tokens per CU.
//
// The activations go through a ring of RING segments, in LDS and in registers: at the start of segment s the
// workgroup writes it to LDS (requested RING segments earlier; at the start all RING at once), requests segment
// s + RING into the registers just freed, and crosses ONE barrier.  A buffer is overwritten RING - 1 barriers
// after its last reader's, so no second barrier is needed.  The weights of a segment, at most 8 steps, are
// requested one segment ahead into one of two register sets; the first set at the very start.
// (The kernel before this one had one segment buffer, two barriers per segment, and the next segment's
// activations in flight for one segment of multiplying, which is shorter than their latency: 768x3072 at 80 %, 333
// tokens with Sum, 15.7 us; 9.9 with 16-token tiles.  The resident kernel of 4096 rows, which the plan takes there, 8.9.)
// =======================================================================================
template <int TM, int OUT, int POST>
struct Ring {
    static constexpr int PIECES = TM / 16, RING = 4, MAXS = SEGMENT_ROWS / STEP_K;
    static constexpr int PASS_ROWS = 512 / PIECES;              // activation rows one load pass of the 512 threads covers
    static constexpr int BUF = SEGMENT_ROWS * TM;
    static constexpr int LDS = RING * BUF + 256;                // activations, then the table
    static constexpr bool TABLE = (POST & SPMM_POST_GELU) != 0 && (OUT == SPMM_OUT_S8 || OUT == SPMM_OUT_U8);

    static __device__ __forceinline__ void run(const Args& a, uint8_t* const lds)
    {
        int tt, rg;
        if (!decode_tile(a, (a.ntiles + 7) / 8, (a.M + TM - 1) / TM, rg, tt)) return;
        const int tid = threadIdx.x;
        const int lane = tid & 63;
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int g = lane >> 4, c = lane & 15;
        const int tok0 = tt * TM;
        const int tile = rg * 8 + wave;
        const bool have_tile = tile < a.ntiles;
        const int n = tile * TILE_ROWS + c;

        // ---- weights of segment s in set s % 2
        v4i A[2][MAXS];
        uint32_t I[2][MAXS];
        auto w_load = [&](v4i (&w)[MAXS], uint32_t (&rows)[MAXS], const int first, const int count) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < MAXS; ++j)
                if (j < count) load_step(a, first + j, lane, w[j], rows[j]);
        };
        // (segment 0 before its bounds have arrived: its first steps follow from tile_steps)
        const bool early = a.tile_steps != 0 && have_tile;
        if (early) w_load(A[0], I[0], tile * a.tile_steps, min(a.tile_steps, MAXS));

        // ---- activations
        v4i xs[RING][PIECES];
        const int x_row = tid / PIECES, x_col = tok0 + tid % PIECES * 16;
        const uint32_t x_lds = Swizzle<TM>::row((uint32_t)x_row) ^ (uint32_t)(tid % PIECES * 16);
        auto x_load = [&](v4i (&x)[PIECES], const int seg) __attribute__((always_inline)) {
            const int k0 = seg * SEGMENT_ROWS, last = min(SEGMENT_ROWS, a.K - k0) - 1;   // rows past K repeat the last one (never multiplied)
            const RaggedPieces<> pieces(a, k0, last);
#pragma unroll
            for (int u = 0; u < PIECES; ++u) x[u] = pieces.load(min(x_row + u * PASS_ROWS, last), x_col);
        };
        auto x_store = [&](v4i (&x)[PIECES], const int buf, const int seg) __attribute__((always_inline)) {
            if (__builtin_expect(tok0 + TM > a.M && a.x_tile_stride == 0, 0)) {
                const int k0 = seg * SEGMENT_ROWS, last = min(SEGMENT_ROWS, a.K - k0) - 1;
                const RaggedPieces<> pieces(a, k0, last);
                if (!pieces.inside) {
#pragma unroll
                    for (int u = 0; u < PIECES; ++u) x[u] = pieces.shifted(x[u], min(x_row + u * PASS_ROWS, last), x_col);
                }
            }
#pragma unroll
            for (int u = 0; u < PIECES; ++u)
                *(v4i*)(lds + buf * BUF + x_lds + u * PASS_ROWS * TM) = x[u] ^ (v4i){FLIP, FLIP, FLIP, FLIP};
        };
#pragma unroll
        for (int q = 0; q < RING; ++q)
            if (q < a.nseg) x_load(xs[q], q);

        // ---- per-row constants, bounds, table, operand of Sum
        const int32_t* const bounds = a.bounds + (int64_t)(have_tile ? tile : 0) * (a.nseg + 1);
        int b0 = 0, b1 = 0, init = 0;                           // steps of the segment about to be multiplied
        float scale = 0.0f, bias = 0.0f;
        if (have_tile) {
            b0 = bounds[0];
            b1 = bounds[1];
            init = a.rowsum[n] * a.corr_mul;
            if (OUT != SPMM_OUT_S32 && n < a.N) {
                scale = a.w_scale[n] * a.x_scale;
                if (a.bias) bias = a.bias[n];
            }
        }
        v4i acc[PIECES];
        v4f sum4[PIECES];
#pragma unroll
        for (int i = 0; i < PIECES; ++i) {
            acc[i] = (v4i){init, init, init, init};
            sum4[i] = (v4f){0.0f, 0.0f, 0.0f, 0.0f};
            const int m0 = tok0 + 16 * i + 4 * g;
            if ((POST & POST_SUM_BIT) && have_tile && n < a.N && m0 < a.M) sum4[i] = load_sum4<POST>(a, n, m0);
        }
        int table_byte = 0;
        if (TABLE && tid < 256) table_byte = a.lut[tid];
        if (!early && have_tile) w_load(A[0], I[0], b0, b1 - b0);
        if (TABLE && tid < 256) lds[RING * BUF + tid] = (uint8_t)table_byte;

        for (int seg0 = 0; seg0 < a.nseg; seg0 += RING) {
#pragma unroll
            for (int q = 0; q < RING; ++q) {
                const int seg = seg0 + q;
                if (seg < a.nseg) {
                    x_store(xs[q], q, seg);
                    int b2 = b1;
                    if (have_tile && seg + 1 < a.nseg) {
                        b2 = bounds[seg + 2];
                        w_load(A[(q + 1) & 1], I[(q + 1) & 1], b1, b2 - b1);
                    }
                    // (behind the weights: loads complete in order, and those are needed first)
                    if (seg + RING < a.nseg) x_load(xs[q], seg + RING);
                    __syncthreads();
#pragma unroll
                    for (int j = 0; j < MAXS; ++j) {
                        if (j < b1 - b0) {
                            const uint32_t o0 = Swizzle<TM>::row(first_row(I[q & 1][j])) + (c & 1) * 8 + q * BUF;
                            const uint32_t o1 = Swizzle<TM>::row(second_row(I[q & 1][j])) + (c & 1) * 8 + q * BUF;
#pragma unroll
                            for (int i = 0; i < PIECES; ++i) {
                                const v2i x0 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i_ptr)(lds + (o0 ^ 16 * i)));
                                const v2i x1 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i_ptr)(lds + (o1 ^ 16 * i)));
                                const v4i xa = {x0[0], x0[1], x1[0], x1[1]};
                                acc[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xa, A[q & 1][j], acc[i], 0, 0, 0);
                            }
                        }
                    }
                    b0 = b1;
                    b1 = b2;
                }
            }
        }

        const LdsTable lut{lds + RING * BUF};
        if (have_tile && n < a.N) {
#pragma unroll
            for (int i = 0; i < PIECES; ++i) {
                const int m0 = tok0 + 16 * i + 4 * g;
                if (m0 < a.M) finish4<OUT, POST, true>(a, acc[i], scale, bias, n, m0, lut, sum4[i]);
            }
        }
    }
};

template <int TM, int NW, int R, int OUT, int POST>
__global__ void __launch_bounds__(512) spmm_rowtile_mfma_simple(const KernelArgs args)
{
    static_assert(NW == 8, "8 waves");
    using Body = Resident<TM, R, TM == 64 ? 1024 : 2048, OUT, POST>;
    __shared__ __attribute__((aligned(16))) uint8_t lds[Body::LDS];
    Body::run(unpack<OUT>(args), lds);
}

template <int TM, int NW, int OUT, int POST>
__global__ void __launch_bounds__(512) spmm_rowtile_mfma_slab(const KernelArgs args)
{
    static_assert(NW == 8, "8 waves");
    using Body = std::conditional_t<TM == 16, Resident<16, 1, SLAB_SEGMENTS * SEGMENT_ROWS, OUT, POST>, Ring<TM, OUT, POST>>;
    __shared__ __attribute__((aligned(16))) uint8_t lds[Body::LDS];
    Body::run(unpack<OUT>(args), lds);
}

template <int TM, int NW, int OUT, int POST>
__global__ void __launch_bounds__(512) spmm_rowtile_mfma_stream(const KernelArgs args)
{
    static_assert(NW == 8, "8 waves");
    using Body = Ring<TM, OUT, POST>;
    __shared__ __attribute__((aligned(16))) uint8_t lds[Body::LDS];
    Body::run(unpack<OUT>(args), lds);
}

}  // namespace spmm
