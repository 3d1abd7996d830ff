// One kernel configuration of the SpMM kernels: this file is compiled once per configuration
// (see build.py), so that the instantiations build in parallel.
//   pipelined kernel : -DSPMM_CFG_TM=<128|96> -DSPMM_CFG_NW=<16|8> -DSPMM_CFG_MAXS=<4|5|6|8>
//   simple kernel    : -DSPMM_CFG_SIMPLE=<1|2> (row tiles per wave) -DSPMM_CFG_SIMPLE_TM=<64|32|16> (token tile)
//   short-batch kernel: -DSPMM_CFG_SLAB=<16|32>      (token tile)
//   streamed kernel  : -DSPMM_CFG_STREAM=<64|32|16>  (token tile)
//   persistent kernel over the wide form: -DSPMM_CFG_WIDE_TM=<128|96|64> -DSPMM_CFG_NW=8, or <64|32> and 4, -DSPMM_CFG_MAXS=<5|6|7|8>
//   loader-fed pipelined kernel: -DSPMM_CFG_FED_TM=<128|96|64> -DSPMM_CFG_NW=<12|8> -DSPMM_CFG_MAXS=<4|6|8>
// Each defines one function launch_cfg_<...>() that picks the epilogue instantiation and
// launches it; spmm_plan.hip calls them.
#if defined(SPMM_CFG_WIDE_TM)
#include "spmm_wide.h"
#else
#include "spmm_kernels.h"
#endif

namespace spmm {

// By its address: <<<>>> has the runtime keep grid and block on a stack first, and takes them back in a stub, with which launches
// back to back take 2.88 us of the host instead of 2.75, and short ones are bound by that (256x256 at 90 %, 128 tokens, called from
// Python: 3.39 and 3.25 us).
template <typename Kernel>
static void launch(Kernel* kernel, dim3 grid, dim3 block, hipStream_t st, const KernelArgs& a)
{
    const void* args[] = {&a};
    (void)hipLaunchKernel((const void*)kernel, grid, block, (void**)args, 0, st);     // (the caller asks for the error)
}

// postop: SPMM_POST_NONE / SPMM_POST_GELU, plus POST_SUM_BIT (combinations the host has
// checked: no Sum with S32 output or with the table chain)
template <class L>
static void dispatch_epilogue(spmm_out_t out_type, int postop, dim3 grid, dim3 block, hipStream_t st,
                              const KernelArgs& a)
{
    const bool gelu = (postop & SPMM_POST_GELU) != 0, sum = (postop & POST_SUM_BIT) != 0;
    constexpr int NONE = SPMM_POST_NONE, GELU = SPMM_POST_GELU, SUM = POST_SUM_BIT;
    switch (out_type) {
    case SPMM_OUT_S32: L::template go<SPMM_OUT_S32, NONE>(grid, block, st, a); break;
    case SPMM_OUT_F32:
        if (gelu && sum) L::template go<SPMM_OUT_F32, GELU | SUM>(grid, block, st, a);
        else if (gelu) L::template go<SPMM_OUT_F32, GELU>(grid, block, st, a);
        else if (sum) L::template go<SPMM_OUT_F32, NONE | SUM>(grid, block, st, a);
        else L::template go<SPMM_OUT_F32, NONE>(grid, block, st, a);
        break;
    case SPMM_OUT_S8:
        if (gelu) L::template go<SPMM_OUT_S8, GELU>(grid, block, st, a);
        else if (sum) L::template go<SPMM_OUT_S8, NONE | SUM>(grid, block, st, a);
        else L::template go<SPMM_OUT_S8, NONE>(grid, block, st, a);
        break;
    case SPMM_OUT_U8:
        if (gelu) L::template go<SPMM_OUT_U8, GELU>(grid, block, st, a);
        else if (sum) L::template go<SPMM_OUT_U8, NONE | SUM>(grid, block, st, a);
        else L::template go<SPMM_OUT_U8, NONE>(grid, block, st, a);
        break;
    }
}

#define SPMM_CAT_(a, b) a##b
#define SPMM_CAT(a, b) SPMM_CAT_(a, b)

// The launcher structs below have the same name in every configuration's object file but launch
// different instantiations: internal linkage keeps the linker from folding their member functions
// into one (which would launch the wrong kernel for every configuration but the one it kept).

#if defined(SPMM_CFG_WIDE_TM)
namespace {
template <int TM, int NW, int MAXS>
struct WideLaunch {
    template <int OUT, int POST>
    static void go(dim3 grid, dim3 block, hipStream_t st, const KernelArgs& a)
    {
        if constexpr (TM <= wide_tile(OUT == SPMM_OUT_F32 && (POST & SPMM_POST_GELU), POST & POST_SUM_BIT))
            launch(spmm_rowtile_smfmac<TM, NW, MAXS, OUT, POST>, grid, block, st, a);
    }
};
}  // namespace

void SPMM_CAT(SPMM_CAT(SPMM_CAT(SPMM_CAT(SPMM_CAT(launch_cfg_wide_, SPMM_CFG_WIDE_TM), _), SPMM_CFG_NW), _), SPMM_CFG_MAXS)(
    spmm_out_t out_type, int postop, const unsigned* grid, unsigned block, void* stream, const KernelArgs& a)
{
    dispatch_epilogue<WideLaunch<SPMM_CFG_WIDE_TM, SPMM_CFG_NW, SPMM_CFG_MAXS>>(out_type, postop, dim3(grid[0], grid[1], grid[2]), dim3(block),
                                                                   (hipStream_t)stream, a);
}
#elif defined(SPMM_CFG_FED_TM)
namespace {
template <int TM, int NW, int MAXS>
struct FedLaunch {
    template <int OUT, int POST>
    static void go(dim3 grid, dim3 block, hipStream_t st, const KernelArgs& a)
    {
        launch(spmm_rowtile_mfma_fed<TM, NW, 4, MAXS, OUT, POST>, grid, block, st, a);
    }
};
}  // namespace

void SPMM_CAT(SPMM_CAT(SPMM_CAT(SPMM_CAT(SPMM_CAT(launch_cfg_fed_, SPMM_CFG_FED_TM), _), SPMM_CFG_NW), _), SPMM_CFG_MAXS)(
    spmm_out_t out_type, int postop, const unsigned* grid, unsigned block, void* stream, const KernelArgs& a)
{
    dispatch_epilogue<FedLaunch<SPMM_CFG_FED_TM, SPMM_CFG_NW, SPMM_CFG_MAXS>>(out_type, postop, dim3(grid[0], grid[1], grid[2]),
                                                                               dim3(block), (hipStream_t)stream, a);
}
#elif defined(SPMM_CFG_STREAM)
namespace {
struct StreamLaunch {
    template <int OUT, int POST>
    static void go(dim3 grid, dim3 block, hipStream_t st, const KernelArgs& a)
    {
        launch(spmm_rowtile_mfma_stream<SPMM_CFG_STREAM, 8, OUT, POST>, grid, block, st, a);
    }
};
}  // namespace

void SPMM_CAT(launch_cfg_stream, SPMM_CFG_STREAM)(spmm_out_t out_type, int postop, const unsigned* grid, unsigned block, void* stream, const KernelArgs& a)
{
    dispatch_epilogue<StreamLaunch>(out_type, postop, dim3(grid[0], grid[1], grid[2]), dim3(block), (hipStream_t)stream, a);
}
#elif defined(SPMM_CFG_SLAB)
namespace {
struct SlabLaunch {
    template <int OUT, int POST>
    static void go(dim3 grid, dim3 block, hipStream_t st, const KernelArgs& a)
    {
        launch(spmm_rowtile_mfma_slab<SPMM_CFG_SLAB, 8, OUT, POST>, grid, block, st, a);
    }
};
}  // namespace

void SPMM_CAT(launch_cfg_slab, SPMM_CFG_SLAB)(spmm_out_t out_type, int postop, const unsigned* grid, unsigned block, void* stream,
                     const KernelArgs& a)
{
    dispatch_epilogue<SlabLaunch>(out_type, postop, dim3(grid[0], grid[1], grid[2]), dim3(block), (hipStream_t)stream, a);
}
#elif defined(SPMM_CFG_SIMPLE)
#ifndef SPMM_CFG_SIMPLE_TM
#define SPMM_CFG_SIMPLE_TM 64
#endif

namespace {
template <int R>
struct SimpleLaunch {
    template <int OUT, int POST>
    static void go(dim3 grid, dim3 block, hipStream_t st, const KernelArgs& a)
    {
        launch(spmm_rowtile_mfma_simple<SPMM_CFG_SIMPLE_TM, 8, R, OUT, POST>, grid, block, st, a);
    }
};
}  // namespace

void SPMM_CAT(SPMM_CAT(SPMM_CAT(launch_cfg_simple_, SPMM_CFG_SIMPLE_TM), _), SPMM_CFG_SIMPLE)(
    spmm_out_t out_type, int postop, const unsigned* grid, unsigned block, void* stream, const KernelArgs& a)
{
    dispatch_epilogue<SimpleLaunch<SPMM_CFG_SIMPLE>>(out_type, postop, dim3(grid[0], grid[1], grid[2]), dim3(block),
                                                     (hipStream_t)stream, a);
}
#else
namespace {
template <int TM, int NW, int MAXS>
struct PipeLaunch {
    template <int OUT, int POST>
    static void go(dim3 grid, dim3 block, hipStream_t st, const KernelArgs& a)
    {
        // one instantiation per layout of the activations and of 1-byte outputs (row-major / token-tile-major):
        // the 16-wave forms have no register to spare for a choice at run time
        const int layout = ((a.k_flags & ARG_X_TILED) ? 1 : 0) | ((a.k_flags & ARG_OUT_TILED) ? 2 : 0);
        if constexpr (OUT == SPMM_OUT_S8 || OUT == SPMM_OUT_U8) {
            if (layout == 3) { launch(spmm_rowtile_mfma<TM, NW, MAXS, OUT, POST, 3>, grid, block, st, a); return; }
            if (layout == 2) { launch(spmm_rowtile_mfma<TM, NW, MAXS, OUT, POST, 2>, grid, block, st, a); return; }
        }
        if (layout & 1) launch(spmm_rowtile_mfma<TM, NW, MAXS, OUT, POST, 1>, grid, block, st, a);
        else launch(spmm_rowtile_mfma<TM, NW, MAXS, OUT, POST, 0>, grid, block, st, a);
    }
};
}  // namespace

void SPMM_CAT(SPMM_CAT(SPMM_CAT(SPMM_CAT(SPMM_CAT(launch_cfg_, SPMM_CFG_TM), _), SPMM_CFG_NW), _), SPMM_CFG_MAXS)(
    spmm_out_t out_type, int postop, const unsigned* grid, unsigned block, void* stream, const KernelArgs& a)
{
    dispatch_epilogue<PipeLaunch<SPMM_CFG_TM, SPMM_CFG_NW, SPMM_CFG_MAXS>>(out_type, postop, dim3(grid[0], grid[1], grid[2]),
                                                                            dim3(block), (hipStream_t)stream, a);
}
#endif

}  // namespace spmm
