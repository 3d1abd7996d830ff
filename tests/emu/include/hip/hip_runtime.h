// Stand-in for <hip/hip_runtime.h> that lets the library's HIP sources compile for the HOST, so that
// the kernels can run on the CPU under memory checks (test infrastructure; never part of the product).
// Every GPU thread is a fiber, a workgroup runs on one OS thread, workgroups run on a few OS threads;
// the cross-lane instructions the kernels use (transposing LDS read, matrix instruction, lane reads,
// lane-row swaps) are emulated by exchanging operands between the 64 fibers of a wave.  Device memory
// is host memory fenced by protected pages: an access outside an allocation is a segmentation fault
// at the faulting kernel line.  A barrier that not every wave of a workgroup reaches is reported as a
// deadlock instead of hanging.
#pragma once
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <algorithm>
#include <functional>
#include <type_traits>

#define __global__
#define __device__
#define __host__
#define __forceinline__ inline __attribute__((always_inline))
#define __launch_bounds__(...)
#define __shared__ static thread_local

struct dim3 {
    unsigned x, y, z;
    dim3(unsigned x_ = 1, unsigned y_ = 1, unsigned z_ = 1) : x(x_), y(y_), z(z_) {}
};
struct float2 { float x, y; };
static inline float2 make_float2(float x, float y) { return float2{x, y}; }

typedef int hipError_t;
typedef void* hipStream_t;
enum { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorOutOfMemory = 2 };
enum { hipMemcpyHostToDevice = 1, hipMemcpyDeviceToHost = 2 };
enum { hipDeviceAttributeMultiprocessorCount = 1 };

namespace emu {
typedef int v4i_t __attribute__((ext_vector_type(4)));
typedef int v2i_t __attribute__((ext_vector_type(2)));
struct Fiber;
Fiber* cur();
dim3& thread_idx();
dim3& block_idx();
dim3& grid_dim();
dim3& block_dim();
void syncthreads();
v2i_t tr8(const void* p);
v4i_t mfma_i8_16x16x64(v4i_t a, v4i_t b, v4i_t c);
typedef int v8i_t __attribute__((ext_vector_type(8)));
typedef int v16i_t __attribute__((ext_vector_type(16)));
v16i_t smfmac_i8_32x32x64(v4i_t a, v8i_t b, v16i_t c, int sel);
void sleep();
int dpp(int v, int control);
int readfirstlane(int v);
void wave_barrier();
void released();
unsigned count_up(unsigned* p, unsigned v, int order);
typedef unsigned v2u_t __attribute__((ext_vector_type(2)));
v2u_t permlane_swap(unsigned a, unsigned b, int rows);
int readlane(int v, int lane);
uint64_t ballot(bool v);
void launch(dim3 grid, dim3 block, const std::function<void()>& fn);
void* dev_alloc(size_t bytes);
void dev_free(void* p);
extern unsigned failing_mallocs;        // bit i: the i-th hipMalloc from here on finds no memory
extern unsigned failing_copies;         // bit i: the i-th hipMemcpy does not (for what it copies through)
extern thread_local int last_error;     // as the runtime keeps it: of the last call that failed, until it is asked for
}  // namespace emu

#define threadIdx (emu::thread_idx())
#define blockIdx (emu::block_idx())
#define gridDim (emu::grid_dim())
#define blockDim (emu::block_dim())
#define __syncthreads() emu::syncthreads()

#define __builtin_amdgcn_readfirstlane(v) emu::readfirstlane((int)(v))
#define __builtin_amdgcn_readlane(v, l) emu::readlane((int)(v), (int)(l))
#define __builtin_amdgcn_ballot_w64(v) emu::ballot(v)
#define __builtin_amdgcn_ds_read_tr8_b64_v2i32(p) emu::tr8((const void*)(uintptr_t)(p))
#define __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, x, y, z) emu::mfma_i8_16x16x64((a), (b), (c))
#define __builtin_amdgcn_smfmac_i32_32x32x64_i8(a, b, c, sel, x, y) emu::smfmac_i8_32x32x64((a), (b), (c), (sel))
#define __builtin_amdgcn_mov_dpp(v, control, rows, banks, bound) emu::dpp((v), (control))
#define __builtin_amdgcn_wave_barrier() emu::wave_barrier()
// (what a wave read or wrote in LDS before a release fence is over when it counts up after it: see count_up)
#define __builtin_amdgcn_fence(order, ...) ((order) == __ATOMIC_RELEASE ? emu::released() : (void)0)
#define __builtin_amdgcn_s_sleep(n) emu::sleep()
#define __builtin_amdgcn_sched_barrier(m) ((void)0)
#define __builtin_amdgcn_permlane16_swap(a, b, fi, bc) emu::permlane_swap((a), (b), 16)
#define __builtin_amdgcn_permlane32_swap(a, b, fi, bc) emu::permlane_swap((a), (b), 32)
#define __builtin_amdgcn_sched_group_barrier(a, b, c) ((void)0)
#define __builtin_amdgcn_s_waitcnt(m) ((void)0)
#define __builtin_amdgcn_s_setprio(m) ((void)0)
#define __builtin_amdgcn_rcpf(x) (1.0f / (x))
#define __builtin_amdgcn_exp2f(x) exp2f(x)
#define __fmaf_rn(a, b, c) fmaf((a), (b), (c))
static inline float emu_fmed3f(float a, float b, float c)
{
    if (a != a || b != b || c != c) return fminf(fminf(a, b), c);
    return fmaxf(fminf(a, b), fminf(fmaxf(a, b), c));
}
#define __builtin_amdgcn_fmed3f(a, b, c) emu_fmed3f((a), (b), (c))
static inline uint32_t emu_cvt_pk_u8_f32(float f, uint32_t sel, uint32_t old)
{
    int v = 0;
    if (f == f) { float r = nearbyintf(f); v = r < 0.0f ? 0 : (r > 255.0f ? 255 : (int)r); }
    const uint32_t sh = 8 * (sel & 3);
    return (old & ~(0xffu << sh)) | ((uint32_t)v << sh);
}
#define __builtin_amdgcn_cvt_pk_u8_f32(f, sel, old) emu_cvt_pk_u8_f32((f), (sel), (old))
static inline uint32_t emu_perm(uint32_t hi, uint32_t lo, uint32_t sel)
{
    const uint64_t v = ((uint64_t)hi << 32) | lo;
    uint32_t r = 0;
    for (int i = 0; i < 4; ++i) {
        const uint32_t s = sel >> (8 * i) & 0xff;
        r |= (s < 8 ? (uint32_t)(v >> (8 * s)) & 0xff : 0u) << (8 * i);      // (0x0c: zero; the kernels use no other)
    }
    return r;
}
#define __builtin_amdgcn_perm(hi, lo, sel) emu_perm((hi), (lo), (sel))
static inline uint32_t emu_alignbyte(uint32_t hi, uint32_t lo, uint32_t sh)
{
    const uint64_t v = ((uint64_t)hi << 32) | lo;
    return (uint32_t)(v >> (8 * (sh & 3)));
}
#define __builtin_amdgcn_alignbyte(hi, lo, sh) emu_alignbyte((hi), (lo), (sh))
// buffer resource + raw buffer store: base pointer and size.  The hardware drops a store that would leave the
// buffer; the kernels never rely on that, so here it ends the run with a message
struct emu_buffer_rsrc { uint8_t* base; uint32_t bytes; };
typedef emu_buffer_rsrc __amdgpu_buffer_rsrc_t;
#define __builtin_amdgcn_make_buffer_rsrc(p, stride, num, flags) (emu_buffer_rsrc{(uint8_t*)(p), (uint32_t)(num)})
template <typename V>
static inline void emu_buffer_store(const V v, const emu_buffer_rsrc r, const int voff, const int soff)
{
    const uint64_t off = (uint64_t)(uint32_t)voff + (uint32_t)soff;
    if (off + sizeof(V) > r.bytes) {
        fprintf(stderr, "emu: buffer store of %zu bytes at offset %llu leaves the buffer of %u bytes\n", sizeof(V),
                (unsigned long long)off, r.bytes);
        abort();
    }
    memcpy(r.base + off, &v, sizeof(V));
}
#define __builtin_amdgcn_raw_buffer_store_b128(v, r, vo, so, aux) emu_buffer_store((v), (r), (vo), (so))
#define __builtin_amdgcn_raw_buffer_store_b32(v, r, vo, so, aux) emu_buffer_store((v), (r), (vo), (so))
// ... and loads, which are zero beyond the end (whole dwords: the kernels' are aligned)
template <typename V>
static inline V emu_buffer_load(const emu_buffer_rsrc r, const int voff, const int soff)
{
    const uint64_t off = (uint64_t)(uint32_t)voff + (uint32_t)soff;
    V v = {};
    for (size_t i = 0; i < sizeof(V); i += 4)
        if (off + i + 4 <= r.bytes) memcpy((uint8_t*)&v + i, r.base + off + i, 4);
    return v;
}
typedef unsigned int emu_v4u __attribute__((vector_size(16)));
#define __builtin_amdgcn_raw_buffer_load_b128(r, vo, so, aux) emu_buffer_load<emu_v4u>((r), (vo), (so))
#define __builtin_amdgcn_raw_buffer_load_b32(r, vo, so, aux) emu_buffer_load<uint32_t>((r), (vo), (so))
using std::min;
using std::max;

static inline hipError_t hipMalloc(void** p, size_t n)
{
    const bool fails = emu::failing_mallocs & 1;
    emu::failing_mallocs >>= 1;
    *p = fails ? nullptr : emu::dev_alloc(n);
    if (!*p) emu::last_error = hipErrorOutOfMemory;
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
static inline hipError_t hipFree(void* p) { emu::dev_free(p); return hipSuccess; }
static inline hipError_t hipMallocAsync(void** p, size_t n, hipStream_t) { return hipMalloc(p, n); }
static inline hipError_t hipFreeAsync(void* p, hipStream_t) { return hipFree(p); }
static inline hipError_t hipMemset(void* p, int v, size_t n) { memset(p, v, n); return hipSuccess; }
static inline hipError_t hipMemcpy(void* d, const void* s, size_t n, int)
{
    const bool fails = emu::failing_copies & 1;
    emu::failing_copies >>= 1;
    if (fails) return emu::last_error = hipErrorOutOfMemory;
    memcpy(d, s, n);
    return hipSuccess;
}
static inline hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
static inline hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
static inline hipError_t hipDeviceGetAttribute(int* v, int, int)
{
    const char* e = getenv("EMU_CUS");
    *v = e ? atoi(e) : 256;
    return hipSuccess;
}
static inline hipError_t hipGetLastError()
{
    const hipError_t e = emu::last_error;
    emu::last_error = hipSuccess;
    return e;
}
#define hipLaunchKernelGGL(kernel, grid, block, shmem, stream, ...) \
    emu::launch((grid), (block), [=]() { kernel(__VA_ARGS__); })
// (the kernel as a function and not as an address: build_emu.py)
template <typename A>
static inline hipError_t hipLaunchKernel(void (*kernel)(A), dim3 grid, dim3 block, void** args, size_t, hipStream_t)
{
    const typename std::remove_const<A>::type a = *(const A*)args[0];
    emu::launch(grid, block, [=]() { kernel(a); });
    return hipSuccess;
}
