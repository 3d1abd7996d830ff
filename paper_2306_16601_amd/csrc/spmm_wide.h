// Persistent kernel over the "wide" form of the packed weight (spmm_internal.h): row tiles of 32 output rows, 64 listed k a
// step, held 2 of 4 for the structured-sparse matrix instruction.
//
// What bounds the kernels of 16-row tiles in long batches is the gather: every listed k of every 16 rows is read from LDS
// once, 16 bytes of it for 16 tokens (a ds_read_b64_tr_b8 of a wave, 512 bytes, reads 32 listed k), and with 4x1 blocks at 75 to
// 90 % most of what is read for 16 rows is listed by the next 16 as well.  32 rows share a list here.  Its length grows by less than
// twice (8 block-rows at 90 %: 57 % of all k against 34 % for 4), so that 5 gathers of 32 rows stand for 6 of two times 16;
// and as no row uses more than two of every four slots (the packer sees to that), one v_smfmac_i32_32x32x64_i8 multiplies
// 32 rows x 64 listed k x 32 tokens in the time of the dense instruction of half as many k.  For such a unit (4 gathers, one
// instruction) a CU with 8 waves of nothing else takes 56 cycles; gathers alone 45, the instruction alone 33.  With random
// operands the chip clocks down to 1.8 GHz in this (the instruction alone: 1.5 GHz), so the parts add up more than the cycles say.
//
// Compute waves take one row tile each, in token tiles of TM; half as many waves again stage activations.  Measured, without
// this kernel and with it: 4096x4096 at 70 %, rows uneven by 20 %, 4096 tokens, row-major s8: 79.6 and 54.6 us (75.4 and 53.5 on
// another machine); the two layers 4096x1024 and 1024x4096 at 85 %, 6144 tokens, tile-major codes: 46.9 and 42.9 us (46.6 and
// 42.2); 2048x1024 in 1x4 blocks at 90 %, 1024 tokens, s8: 7.5 and 6.3 us.
#pragma once

#include "spmm_kernels.h"

namespace spmm {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef unsigned int v2u __attribute__((ext_vector_type(2)));
// memory that no kernel writes, read through the scalar unit even behind fences (a vector load in its place was waited for
// with every load before it)
typedef const __attribute__((address_space(4))) int32_t* constant_int_ptr;

// f(0), f(1), .. f(N - 1), each with its number as a constant
template <int N, int I = 0, typename F>
__device__ __forceinline__ void each(const F& f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        each<N, I + 1>(f);
    }
}

// lane I of every 16 lanes, in all of them (DPP row_newbcast)
template <int I>
__device__ __forceinline__ int of_lane(const int v)
{
    return __builtin_amdgcn_mov_dpp(v, 0x150 + I, 0xf, 0xf, true);
}
template <int I>
__device__ __forceinline__ float of_lane(const float v)
{
    return __builtin_bit_cast(float, of_lane<I>(__builtin_bit_cast(int, v)));
}

template <int TM, int NW, int MAXS, int OUT, int POST>
struct Wide {
    static constexpr int LW = NW / 2, THREADS = (NW + LW) * 64, PIECES = TM / 32;
    // a buffer: [piece][512 rows][32 tokens]
    static constexpr int PIECE = SEGMENT_ROWS * 32 + 64, BUF = PIECES * PIECE;
    static constexpr bool BYTES = OUT == SPMM_OUT_S8 || OUT == SPMM_OUT_U8;
    static constexpr bool TABLE = (POST & SPMM_POST_GELU) != 0 && BYTES;
    static constexpr bool SUM = (POST & POST_SUM_BIT) != 0;
    // LDS: table, counts, constants of the rows, buffers, staging of 1-byte outputs.  As many buffers as there is room for, up
    // to four: the waves that go first run ahead by as many phases less one.
    static constexpr int COUNTS = 256, CONSTANTS = COUNTS + 64, X0 = CONSTANTS + NW * 768;
    static constexpr int PAIR = PIECES == 3 ? 1 : 2;        // pieces that 1-byte outputs are staged by
    static constexpr int BUFFERS = TM == 128 || (TM == 64 && NW == 4) ? 2 : TM == 96 ? 3 : 4;
    static constexpr int STAGE = X0 + BUFFERS * BUF, LDS = STAGE + (BYTES ? NW * 1024 * PAIR : 0);
    static_assert(LDS <= 160 * 1024 / (8 / NW), "12 waves per CU");
    static constexpr int AHEAD = PIECES == 4 && MAXS > 6 ? 2 : 3;       // gathers of this many pieces in flight

    // staging, by the loader waves: 16-byte units; UNITS of a row, ROWS_PER_PASS rows of a pass
    static constexpr int UNITS = 2 * PIECES, ROWS_PER_PASS = PIECES == 3 ? 32 : LW * 64 / UNITS, STAGERS = ROWS_PER_PASS * UNITS;
    static constexpr int XLOADS = SEGMENT_ROWS / ROWS_PER_PASS;

    struct Step {
        v4i w;          // the weight operand, 16 stored values
        v2u more;       // which of 4 listed k each of them is; activation rows (times 32) of two of this lane's four gathers
    };
    struct Range { int first, count; };

    static __device__ __forceinline__ void load_step(const Args& a, const int step, const int lane, Step& s)
    {
        const uint8_t* r = a.records + (int64_t)step * WIDE_RECORD_BYTES;
        s.w = *(const v4i*)(r + (uint32_t)lane * 16u);
        s.more = *(const v2u*)(r + (WIDE_VAL_BYTES + (uint32_t)lane * 8u));
    }

    static __device__ __forceinline__ void run(const KernelArgs& args, uint8_t* const lds)
    {
        Args a = unpack<OUT>(args);
        a.ntiles = (a.N + WIDE_ROWS - 1) / WIDE_ROWS;
        a.bounds = (const int32_t*)(args.weight + wide_bounds_offset(a.ntiles));
        a.records = args.weight + wide_records_offset(a.ntiles, a.nseg);
        const int tid = threadIdx.x;
        const int lane = tid & 63;
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

        const int S = a.n_streams;
        int stream, rg;
        if (!decode_workgroup(a, (a.ntiles + NW - 1) / NW, S, rg, stream)) return;
        const int n_my = a.tiles_per_stream + (stream < (a.M + TM - 1) / TM - a.tiles_per_stream * S ? 1 : 0);
        const int total = n_my * a.nseg;
        struct Phase { int seg, tok0; };
        auto after = [&](Phase f) __attribute__((always_inline)) {
            if (++f.seg == a.nseg) { f.seg = 0; f.tok0 += S * TM; }
            return f;
        };
        Phase cur = {0, stream * TM};

        // ---- in step, but not in lock-step.  The loader waves write phase q's activations over those of phase q - BUFFERS, when all
        // compute waves have multiplied these; a compute wave multiplies phase q when all of its activations are written.
        // Counts of both, for each of four consecutive phases.  The first half of the compute waves (of 8, one on every SIMD; of 4,
        // two of the four SIMDs', the other workgroup's on the others) has priority at first, and so runs ahead of the second,
        // which has it later and ends no later: the post-operators of the one are worked out while the other multiplies.
        unsigned* const counts = (unsigned*)(lds + COUNTS);           // [0 .. 3]: written, [4 .. 7]: multiplied
        constexpr int WRITTEN = 0, MULTIPLIED = 4;
        // (Released on either side: written activations are in LDS, and gathers, also those requested past a segment's last step,
        // have been read, before the count says so.)
        auto signal = [&](const int which, const int q) __attribute__((always_inline)) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_wave_barrier();
            if (lane == 0) __atomic_fetch_add(counts + which + (q & 3), 1u, __ATOMIC_RELAXED);
        };
        auto count = [&](const int which, const int q) __attribute__((always_inline)) {
            return (int)__atomic_load_n(counts + which + (q & 3), __ATOMIC_RELAXED);
        };
        auto wait_for = [&](const int which, const int q, int seen) __attribute__((always_inline)) {
            const int all = (which == WRITTEN ? LW : NW) * (q / 4 + 1);
            while (seen < all) {
                __builtin_amdgcn_s_sleep(1);
                seen = __builtin_amdgcn_readfirstlane(count(which, q));
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        };

        if (wave >= NW) {
            // ------------------------------------------------------------------ loader wave
            const int ltid = tid - NW * 64;
            const bool stager = ltid < STAGERS;
            const int row0 = ltid / UNITS, unit = ltid % UNITS;
            v4i xr[XLOADS];
            auto x_issue = [&]() __attribute__((always_inline)) {       // (and steps to the next phase)
                const int tok0 = cur.tok0, k0 = cur.seg * SEGMENT_ROWS;
                cur = after(cur);
                const int last = min(SEGMENT_ROWS, a.K - k0) - 1;       // rows past K repeat the last one (never multiplied)
                if (!stager) return;
                if (tok0 + TM <= a.M) {
                    const uint8_t* src = a.X + (int64_t)k0 * a.ldx + xcol(a, tok0);
                    const uint32_t ldx = (uint32_t)a.ldx, off = (uint32_t)xcol(a, unit * 16);
                    const uint32_t first = (uint32_t)row0 * ldx + off, end = (uint32_t)last * ldx + off;
#pragma unroll
                    for (int u = 0; u < XLOADS; ++u) xr[u] = load16_any(src + min(first + (uint32_t)(u * ROWS_PER_PASS) * ldx, end));
                } else {
                    const RaggedPieces<> tail(a, k0, last);
                    const int col = tok0 + unit * 16;
#pragma unroll
                    for (int u = 0; u < XLOADS; ++u) xr[u] = tail.load(min(row0 + u * ROWS_PER_PASS, last), col);
                    if (!tail.inside) {
#pragma unroll
                        for (int u = 0; u < XLOADS; ++u) xr[u] = tail.shifted(xr[u], min(row0 + u * ROWS_PER_PASS, last), col);
                    }
                }
            };
            auto x_commit = [&](const int q) __attribute__((always_inline)) {
                if (!stager) return;
                uint8_t* const to = lds + (X0 + q % BUFFERS * BUF) + (row0 * 32 + (unit >> 1) * PIECE + (unit & 1) * 16);
#pragma unroll
                for (int u = 0; u < XLOADS; ++u) *(v4i*)(to + u * ROWS_PER_PASS * 32) = xr[u] ^ (v4i){FLIP, FLIP, FLIP, FLIP};
            };
            if (ltid < 8) counts[ltid] = ltid == 0 ? LW : 0;            // (phase 0's activations are written before the barrier)
            x_issue();
            int table[4 / LW];
            if constexpr (TABLE) {
#pragma unroll
                for (int i = 0; i < 4 / LW; ++i) table[i] = a.lut[i * LW * 64 + ltid];
            }
            x_commit(0);
            if constexpr (TABLE) {
#pragma unroll
                for (int i = 0; i < 4 / LW; ++i) lds[i * LW * 64 + ltid] = (uint8_t)table[i];
            }
            if (1 < total) x_issue();
            __syncthreads();
            for (int q = 1; q < total; ++q) {
                if (q >= BUFFERS) wait_for(MULTIPLIED, q - BUFFERS, 0);
                x_commit(q);
                signal(WRITTEN, q);
                if (q + 1 < total) x_issue();
            }
            return;
        }

        // ---------------------------------------------------------------------- compute wave
        const int tile = rg * NW + wave;
        const bool have_tile = tile < a.ntiles;

        // ---- weights.  One set of registers, requested again in two halves, for the next phase, as soon as they have been
        // multiplied (a set for each of two segments that stay leaves the wider tiles too few registers for the rest).  Slots
        // past a segment's last step hold that step again (their rows are gathered, never multiplied), so that every phase requests
        // the same number of records whatever its length, and a wait for one is not one for all.
        Step w[MAXS];
        v16i acc[PIECES];
        // step ranges of the phases, in order: up to 16 segments' counts, at most 8 each, in a scalar register pair
        const constant_int_ptr bounds = (constant_int_ptr)(uintptr_t)(a.bounds + (int64_t)(have_tile ? tile : 0) * (a.nseg + 1));
        uint64_t counted = 0;
        int w_seg = 0, tile_first = 0, w_first = 0;
        auto next_range = [&]() __attribute__((always_inline)) {
            Range r = {w_first, 0};
            if (have_tile) r.count = a.nseg <= 16 ? (int)(counted >> (4 * w_seg)) & 15 : bounds[w_seg + 1] - bounds[w_seg];
            w_first += r.count;
            if (++w_seg == a.nseg) {
                w_seg = 0;
                w_first = tile_first;
            }
            return r;
        };
        auto w_slot = [&](const Range r, const int s) __attribute__((always_inline)) {
            load_step(a, max(r.first + min(s, r.count - 1), 0), lane, w[s]);
        };

        // ---- multiply phase q (and request weights into the registers that it leaves; and look whether the next one's activations
        // are written)
        auto multiply = [&](const int q, const int cnt, const Range next, int& seen) __attribute__((always_inline)) {
            const int me = pinned(lane);
            const uint32_t base = X0 + (uint32_t)(q % BUFFERS) * BUF + (uint32_t)((me >> 4) & 1) * 16 + (uint32_t)(me & 1) * 8;
            v8i x[AHEAD + 1];
            v2u rows;       // of the step being gathered
            auto gather = [&](const int u) __attribute__((always_inline)) {
                if (u % PIECES == 0) {      // (from the even and the odd lane of a pair)
                    const int pair = pinned((int)w[u / PIECES].more[1]);
                    rows = (v2u){(unsigned)__builtin_amdgcn_mov_dpp(pair, 0xA0, 0xf, 0xf, true),
                                 (unsigned)__builtin_amdgcn_mov_dpp(pair, 0xF5, 0xf, 0xf, true)};
                }
                const int at = (u % PIECES) * PIECE;
                const v2i x0 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i_ptr)(lds + ((rows[0] & 0xffff) + base) + at));
                const v2i x1 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i_ptr)(lds + ((rows[0] >> 16) + base) + at));
                const v2i x2 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i_ptr)(lds + ((rows[1] & 0xffff) + base) + at));
                const v2i x3 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i_ptr)(lds + ((rows[1] >> 16) + base) + at));
                x[u % (AHEAD + 1)] = (v8i){x0[0], x0[1], x1[0], x1[1], x2[0], x2[1], x3[0], x3[1]};
            };
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) gather(u);
            __builtin_amdgcn_sched_barrier(0);
            // (chains that are left at the last step, with no way back in: where paths meet, the compiler has a gather wait for
            // all before it)
            auto steps = [&](auto&& self, auto S, auto END) __attribute__((always_inline)) {
                constexpr int s = S.value;
                if constexpr (s < END.value) {
                    if (s < cnt) {
#pragma unroll
                        for (int i = 0; i < PIECES; ++i) {
                            const int u = s * PIECES + i;
                            if (u + AHEAD < MAXS * PIECES) gather(u + AHEAD);
                            acc[i] = __builtin_amdgcn_smfmac_i32_32x32x64_i8(w[s].w, x[u % (AHEAD + 1)], acc[i], (int)w[s].more[0], 0, 0);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                        self(self, std::integral_constant<int, s + 1>{}, END);
                    }
                }
            };
            steps(steps, std::integral_constant<int, 0>{}, std::integral_constant<int, MAXS / 2>{});
#pragma unroll
            for (int s = 0; s < MAXS / 2; ++s) w_slot(next, s);
            seen = count(WRITTEN, q + 1);
            steps(steps, std::integral_constant<int, MAXS / 2>{}, std::integral_constant<int, MAXS>{});
#pragma unroll
            for (int s = MAXS / 2; s < MAXS; ++s) w_slot(next, s);
            seen = __builtin_amdgcn_readfirstlane(seen);
        };

        // ---- post-operators and stores: lane (h = lane / 32, t = lane % 32) holds, in register 4 q + r of piece i, row
        // 8 q + 4 h + r of the tile and token 32 i + t
        // constants of the rows (correction, scale, bias), in lane 16 g + 4 q + r those of row 8 q + 4 (g / 2) + r
        int32_t* const constants = (int32_t*)(lds + CONSTANTS + wave * 768);
        auto reset = [&]() __attribute__((always_inline)) {
            const int init = constants[pinned(lane)];
            each<16>([&](auto I) {
#pragma unroll
                for (int i = 0; i < PIECES; ++i) acc[i][I.value] = of_lane<I.value>(init);
            });
        };
        const __amdgpu_buffer_rsrc_t rs = out_resource(a);
        auto finish = [&](auto FULL, const int tok0) __attribute__((always_inline)) {
            const int me = pinned(lane), h = me >> 5, t = me & 31;
            const int row0 = tile * WIDE_ROWS;
            const float row_scale = __builtin_bit_cast(float, constants[64 + me]), row_bias = __builtin_bit_cast(float, constants[128 + me]);
            const int g = me >> 4, p = me & 15;
            const uint32_t stage = STAGE + wave * (1024 * PAIR);
            // 16 tokens of a row
            auto store = [&](const int row, const int m, const v4i v) __attribute__((always_inline)) {
                const int n = row0 + row;
                const bool ot = a.out_tile_stride != 0;
                const uint32_t off = ot ? (uint32_t)(m >> 5) * (uint32_t)a.out_tile_stride + (uint32_t)n * 32u + (uint32_t)(m & 31)
                                        : (uint32_t)n * (uint32_t)a.ldo + (uint32_t)m;
                if (FULL.value || (n < a.N && m + 16 <= a.M)) {
                    if (ot) store16_out<SCOPE_AGENT>(rs, off, v);
                    else ((v4i_any*)((uint8_t*)a.out + off))->v = v;
                } else if (n < a.N && m < a.M) {
                    store_cut16((uint8_t*)a.out + off, v, a.M - m);
                }
            };
            // the four rows of q (I = 4 q + r) of pieces i0 and i0 + 1
            auto values = [&](const int i0, auto Q, float (&y)[2][4]) __attribute__((always_inline)) {
                each<4>([&](auto R) {
                    constexpr int I = 4 * Q.value + R.value;
                    const float scale = of_lane<I>(row_scale), bias = of_lane<I>(row_bias);
#pragma unroll
                    for (int i = 0; i < 2; ++i)
                        if (i0 + i < PIECES) {
                            y[i][R.value] = __fmaf_rn((float)acc[i0 + i][I], scale, bias);
                            if constexpr (OUT == SPMM_OUT_F32 && (POST & SPMM_POST_GELU) != 0) y[i][R.value] = gelu_f32(y[i][R.value]);
                        }
                    if constexpr (OUT == SPMM_OUT_F32 && (POST & SPMM_POST_GELU) != 0 && PIECES > 2) __builtin_amdgcn_sched_barrier(0);
                });
            };
            auto load_sum = [&](const int i, const int q, float (&sum)[4]) __attribute__((always_inline)) {
                if constexpr (SUM) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        if constexpr (FULL.value) {
                            const float* const from = a.sum + ((int64_t)(row0 + 8 * q + r) * a.ld_sum + (tok0 + 32 * i));
                            sum[r] = from[(uint32_t)(4 * h) * (uint32_t)a.ld_sum + (uint32_t)t];
                        } else {    // (what is past the end repeats the last value and is not stored)
                            const int n = min(row0 + 8 * q + 4 * h + r, a.N - 1), m = min(tok0 + 32 * i + t, a.M - 1);
                            sum[r] = a.sum[(uint32_t)n * (uint32_t)a.ld_sum + (uint32_t)m];
                        }
                    }
                }
            };
            // codes of two pieces, through the wave's own 2 KB, [piece of two][h][token][4 q + r], so that a lane holds 16 tokens
            // of a row
            auto store_codes = [&](const int i0, const v4i (&codes)[2]) __attribute__((always_inline)) {
                const bool two = PAIR == 2 && i0 + 1 < PIECES;
                *(v4i*)(lds + stage + h * 512 + t * 16) = codes[0];
                if (two) *(v4i*)(lds + stage + 1024 + h * 512 + t * 16) = codes[1];
                const int row = 16 * (p >> 3) + 8 * ((p >> 2) & 1) + (p & 3);
                auto fetch = [&](const uint32_t from) __attribute__((always_inline)) {
                    const v2i lo = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i_ptr)(lds + from));
                    const v2i hi = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i_ptr)(lds + from + 128));
                    return (v4i){lo[0], lo[1], hi[0], hi[1]};
                };
                const uint32_t from = stage + (16 * (g & 1) + (p >> 1)) * 16 + (p & 1) * 8;
                if (two) {
                    const v4i low = fetch(from + (g >> 1) * 1024), high = fetch(from + (g >> 1) * 1024 + 512);
                    store(row, tok0 + 32 * i0 + 16 * g, low);
                    store(row + 4, tok0 + 32 * i0 + 16 * g, high);
                } else {
                    store(row + 4 * (g >> 1), tok0 + 32 * i0 + 16 * (g & 1), fetch(from + (g >> 1) * 512));
                    if (i0 + 1 < PIECES) {
                        *(v4i*)(lds + stage + h * 512 + t * 16) = codes[1];
                        store(row + 4 * (g >> 1), tok0 + 32 * (i0 + 1) + 16 * (g & 1), fetch(from + (g >> 1) * 512));
                    }
                }
            };
            if constexpr (TABLE) {
                // The look-ups of two pieces are under way together: one by one, their latency behind the other waves' gathers
                // was most of the time.
                uint32_t v[2][4][4];
                auto look_up = [&](const int i0) __attribute__((always_inline)) {
                    each<4>([&](auto Q) {
                        float y[2][4];
                        values(i0, Q, y);
#pragma unroll
                        for (int i = 0; i < 2; ++i)
#pragma unroll
                            for (int r = 0; r < 4; ++r)
                                if (i0 + i < PIECES) v[i][Q.value][r] = table_key<true>(y[i][r] * a.inv);
                        if constexpr (PIECES == 4) __builtin_amdgcn_sched_barrier(0);
                    });
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int q = 0; q < 4; ++q)
#pragma unroll
                            for (int r = 0; r < 4; ++r)
                                if (i0 + i < PIECES) v[i][q][r] = lds[v[i][q][r]];
                    __builtin_amdgcn_sched_barrier(0);
                };
#pragma unroll
                for (int i0 = 0; i0 < PIECES; i0 += 2) {
                    look_up(i0);
                    v4i codes[2];
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            if (i0 + i < PIECES) {
                                const uint32_t (&b)[4] = v[i][q];
                                codes[i][q] = (int)(__builtin_amdgcn_perm(b[1], b[0], 0x0c0c0400u) | __builtin_amdgcn_perm(b[3], b[2], 0x04000c0cu));
                            }
                    store_codes(i0, codes);
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {
                // (the operand of Sum one group ahead: a load that follows stores would be waited for with them)
                constexpr int GROUPS = 4 * ((PIECES + 1) / 2);
                float sum[2][2][4];
                auto load_sums = [&](auto G) __attribute__((always_inline)) {
                    if constexpr (SUM && G.value < GROUPS) {
#pragma unroll
                        for (int i = 0; i < 2; ++i)
                            if (G.value / 4 * 2 + i < PIECES) load_sum(G.value / 4 * 2 + i, G.value & 3, sum[G.value & 1][i]);
                    }
                };
                load_sums(std::integral_constant<int, 0>{});
                v4i codes[2];
                each<GROUPS>([&](auto G) {
                    constexpr int i0 = G.value / 4 * 2, q = G.value & 3;
                    load_sums(std::integral_constant<int, G.value + 1>{});
                    float y[2][4];
                    if constexpr (OUT != SPMM_OUT_S32) values(i0, std::integral_constant<int, q>{}, y);
                    uint32_t bits[2][4];
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        if (i0 + i >= PIECES) continue;
                        if constexpr (SUM) {
#pragma unroll
                            for (int r = 0; r < 4; ++r) y[i][r] = y[i][r] + sum[G.value & 1][i][r];
                        }
                        if constexpr (BYTES) {
                            codes[i][q] = (int)quantise4<OUT, POST>(a, y[i], LdsTable{lds});
                        } else {
#pragma unroll
                            for (int r = 0; r < 4; ++r) {
                                if constexpr (OUT == SPMM_OUT_S32) bits[i][r] = (uint32_t)acc[i0 + i][4 * q + r];
                                else bits[i][r] = __builtin_bit_cast(uint32_t, y[i][r]);
                            }
                        }
                    }
                    if constexpr (BYTES) {
                        if constexpr (q == 3) store_codes(i0, codes);
                    } else if constexpr (FULL.value) {
                        // (rows that are not 16-byte aligned: at the default scope, see takes_fast_stores)
                        auto store4 = [&](auto SCOPE) __attribute__((always_inline)) {
#pragma unroll
                            for (int r = 0; r < 4; ++r)
#pragma unroll
                                for (int i = 0; i < 2; ++i)
                                    if (i0 + i < PIECES) {
                                        const uint32_t off = 4u * ((uint32_t)(4 * h) * (uint32_t)a.ldo + (uint32_t)t) + 128u * (i0 + i);
                                        __builtin_amdgcn_raw_buffer_store_b32(bits[i][r], rs, (int)off,
                                                                              (int)(4u * ((uint32_t)(row0 + 8 * q + r) * (uint32_t)a.ldo + (uint32_t)tok0)), SCOPE.value);
                                    }
                        };
                        if (a.out_aligned) store4(std::integral_constant<int, SCOPE_AGENT>{});
                        else store4(std::integral_constant<int, SCOPE_DEFAULT>{});
                    } else {
#pragma unroll
                        for (int i = 0; i < 2; ++i)
#pragma unroll
                            for (int r = 0; r < 4; ++r) {
                                const int n = row0 + 8 * q + r + 4 * h, m = tok0 + 32 * (i0 + i) + t;
                                if (i0 + i < PIECES && n < a.N && m < a.M) ((uint32_t*)a.out)[(uint32_t)n * (uint32_t)a.ldo + (uint32_t)m] = bits[i][r];
                            }
                    }
                    if constexpr (PIECES > 2 || SUM || q == 3) __builtin_amdgcn_sched_barrier(0);
                });
            }
        };

        // ---- start-up: the first steps' weights, the constants of the rows; the other weights when the first activations,
        // which share the way into the CU with them, have arrived
        constexpr int FIRST = 2;
        Range early = {0, 0};
        if (have_tile && a.tile_steps) early = {tile * a.tile_steps, a.tile_steps};
        if (have_tile && !a.tile_steps) early = {bounds[0], bounds[1] - bounds[0]};
#pragma unroll
        for (int s = 0; s < FIRST; ++s) w_slot(early, s);
        {
            const int n = tile * WIDE_ROWS + 8 * (lane >> 2 & 3) + 4 * (lane >> 5) + (lane & 3);
            int init = 0;
            float scale = 0.0f, bias = 0.0f;
            if (have_tile) init = a.rowsum[n] * a.corr_mul;
            if (OUT != SPMM_OUT_S32 && have_tile && n < a.N) {
                scale = a.w_scale[n] * a.x_scale;
                if (a.bias) bias = a.bias[n];
            }
            constants[lane] = init;
            constants[64 + lane] = __builtin_bit_cast(int32_t, scale);
            constants[128 + lane] = __builtin_bit_cast(int32_t, bias);
        }
        if (have_tile) {
            const int bound = a.bounds[(int64_t)tile * (a.nseg + 1) + min(lane, a.nseg)];
            w_first = tile_first = __builtin_amdgcn_readlane(bound, 0);
            each<16>([&](auto I) {
                if (I.value < a.nseg)
                    counted |= (uint64_t)(__builtin_amdgcn_readlane(bound, I.value + 1) - __builtin_amdgcn_readlane(bound, I.value)) << (4 * I.value);
            });
        }
        Range here = next_range(), next = next_range();
        __syncthreads();
#pragma unroll
        for (int s = FIRST; s < MAXS; ++s) w_slot(here, s);
        reset();
        int seen = 0;
        const int turn = n_my > 1 ? a.nseg : (total + 1) / 2;
        for (int p = 0; p < total; ++p) {
            const Phase at = cur;
            cur = after(cur);
            if (p > 0) wait_for(WRITTEN, p, seen);
            if (p == 0 || p == turn) {
                if ((wave < NW / 2) == (p < turn)) __builtin_amdgcn_s_setprio(1);
                else __builtin_amdgcn_s_setprio(0);
            }
            multiply(p, here.count, next, seen);
            if (p + BUFFERS < total) signal(MULTIPLIED, p);
            here = next;
            next = next_range();
            if (at.seg == a.nseg - 1 && have_tile) {
                if (at.tok0 + TM <= a.M && (tile + 1) * WIDE_ROWS <= a.N) finish(std::true_type{}, at.tok0);
                else finish(std::false_type{}, at.tok0);
                if (p + 1 < total) reset();
            }
        }
    }
};

template <int TM, int NW, int MAXS, int OUT, int POST>
__global__ void __launch_bounds__(NW * 96, 3) spmm_rowtile_smfmac(const KernelArgs args)
{
    using Body = Wide<TM, NW, MAXS, OUT, POST>;
    __shared__ __attribute__((aligned(16))) uint8_t lds[Body::LDS];
    Body::run(args, lds);
}

}  // namespace spmm
