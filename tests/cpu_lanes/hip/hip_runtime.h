// Stands in for the HIP headers where a kernel source is compiled for the CPU by
// the tests: the lanes of a workgroup are fibers that take turns, and whatever
// lanes exchange (ballots, lane reads, barriers) waits until every live lane of
// the wavefront or workgroup has arrived. Device memory is host memory between
// two inaccessible pages. It covers what the window pass, the split search and
// the profile loader use, and nothing else.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>

using std::max;
using std::min;

#define __global__
#define __device__
#define __host__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __align__(n) __attribute__((aligned(n)))
#define __shared__ static        // "extern __shared__" becomes "extern" when the source is copied

struct alignas(8) uint2 { uint32_t x, y; };
struct alignas(16) uint4 { uint32_t x, y, z, w; };
struct alignas(16) longlong2 { long long x, y; };
inline uint2 make_uint2(uint32_t x, uint32_t y) { return {x, y}; }
struct dim3 {
    unsigned x, y, z;
    dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};

namespace lanes {

extern dim3 thread_idx, block_idx, block_dim, grid_dim;
extern int cus, max_lds;                                       // the device the host code sees
void launch(dim3 grid, dim3 block, size_t lds, const std::function<void()> &kernel);
const uint64_t *exchange(uint64_t v, uint64_t *present);       // every lane's value, and which lanes are there
void sync_block();
void broken(const char *what, const char *file, int line);     // a condition that the source states does not hold
void *device_alloc(size_t bytes);
void device_free(void *p);

inline int lane() { return thread_idx.x & 63; }
inline uint64_t ballot(bool c)
{
    uint64_t there;
    const uint64_t *v = exchange(c, &there);
    uint64_t m = 0;
    for (int i = 0; i < 64; i++)
        if (((there >> i) & 1) && v[i]) m |= uint64_t(1) << i;
    return m;
}
inline int read_lane(int v, int l)
{
    uint64_t there;
    return (int)(uint32_t)exchange((uint32_t)v, &there)[l & 63];
}
inline int read_first(int v)
{
    uint64_t there;
    const uint64_t *e = exchange((uint32_t)v, &there);
    return (int)(uint32_t)e[__builtin_ctzll(there)];
}
// quad_perm, row_shr 1 .. 15, mirrors of 16 and 8 lanes, row_bcast 15 and 31
inline int update_dpp(int old, int v, int ctrl, int row_mask)
{
    uint64_t there;
    const uint64_t *e = exchange((uint32_t)v, &there);
    const int l = lane(), row = l >> 4;
    if (!((row_mask >> row) & 1)) return old;
    int from = -1;
    if (ctrl < 0x100) from = (l & ~3) + ((ctrl >> (2 * (l & 3))) & 3);
    else if (ctrl == 0x140 || ctrl == 0x141) from = l ^ (ctrl == 0x140 ? 15 : 7);
    else if (ctrl > 0x110 && ctrl < 0x120) from = (l & 15) >= ctrl - 0x110 ? l - (ctrl - 0x110) : -1;
    else if (ctrl == 0x142) from = row ? row * 16 - 1 : -1;
    else if (ctrl == 0x143) from = row >= 2 ? 31 : -1;
    else abort();
    return from < 0 ? old : (int)(uint32_t)e[from];
}
template <class T> T shfl_xor(T v, int o)
{
    uint64_t bits = 0, there;
    memcpy(&bits, &v, sizeof(T));
    const uint64_t r = exchange(bits, &there)[lane() ^ o];
    T u;
    memcpy(&u, &r, sizeof(T));
    return u;
}
template <class T, class U> T atomic_add(T *p, U v)
{
    const T old = *p;
    *p += (T)v;
    return old;
}

}  // namespace lanes

#define HEDDLE_INVARIANT(c) ((c) ? (void)0 : lanes::broken(#c, __FILE__, __LINE__))

#define threadIdx lanes::thread_idx
#define blockIdx lanes::block_idx
#define blockDim lanes::block_dim
#define gridDim lanes::grid_dim
#define __syncthreads lanes::sync_block
#define __lane_id lanes::lane
#define __shfl_xor lanes::shfl_xor
#define atomicAdd lanes::atomic_add
#define __clzll(x) __builtin_clzll(x)
#define __umul24(a, b) (((a) & 0xFFFFFFu) * ((b) & 0xFFFFFFu))
#define __popcll(x) __builtin_popcountll(x)
#define __builtin_amdgcn_fence(...) ((void)0)
#define __builtin_amdgcn_wave_barrier() ((void)lanes::ballot(true))
#define __builtin_amdgcn_ballot_w64 lanes::ballot
#define __builtin_amdgcn_readlane lanes::read_lane
#define __builtin_amdgcn_readfirstlane lanes::read_first
#define __builtin_amdgcn_update_dpp(old, v, ctrl, rm, bm, bc) lanes::update_dpp(old, v, ctrl, rm)
#define __builtin_amdgcn_mov_dpp(v, ctrl, rm, bm, bc) lanes::update_dpp(0, v, ctrl, rm)
#define __builtin_amdgcn_mbcnt_lo(m, b) ((b) + (uint32_t)__builtin_popcount((m) & (lanes::lane() < 32 ? (1u << lanes::lane()) - 1 : ~0u)))
#define __builtin_amdgcn_mbcnt_hi(m, b) ((b) + (uint32_t)__builtin_popcount((m) & (lanes::lane() < 32 ? 0u : (1u << (lanes::lane() - 32)) - 1)))
inline float __uint_as_float(uint32_t v) { float f; memcpy(&f, &v, 4); return f; }

// ---- the host interface
typedef int hipError_t;
enum { hipSuccess = 0, hipErrorOutOfMemory = 2, hipErrorInvalidDevice = 101 };
typedef struct ihipStream_t *hipStream_t;
typedef struct ihipEvent_t *hipEvent_t;
typedef struct ihipMemPool_t *hipMemPool_t;
struct hipMemPoolProps { int allocType; struct { int type, id; } location; };
enum { hipMemAllocationTypePinned, hipMemLocationTypeDevice, hipMemPoolAttrReleaseThreshold, hipEventDisableTiming,
       hipMemcpyHostToDevice, hipFuncAttributeMaxDynamicSharedMemorySize, hipDeviceAttributeMultiprocessorCount,
       hipDeviceAttributeMaxSharedMemoryPerBlock, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor };
#define hipStreamPerThread ((hipStream_t)2)
inline const char *hipGetErrorString(hipError_t) { return "error"; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
inline hipError_t hipSetDevice(int) { return hipSuccess; }
inline hipError_t hipStreamGetDevice(hipStream_t, int *d) { *d = 0; return hipSuccess; }
inline hipError_t hipMemPoolCreate(hipMemPool_t *, const hipMemPoolProps *) { return hipSuccess; }
inline hipError_t hipMemPoolSetAttribute(hipMemPool_t, int, void *) { return hipSuccess; }
inline hipError_t hipMemPoolDestroy(hipMemPool_t) { return hipSuccess; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t *, unsigned) { return hipSuccess; }
inline hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
inline hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
inline hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
inline hipError_t hipDeviceSynchronize() { return hipSuccess; }
inline hipError_t hipMalloc(void *p, size_t n) { *(void **)p = lanes::device_alloc(n); return hipSuccess; }
inline hipError_t hipFree(void *p) { lanes::device_free(p); return hipSuccess; }
inline hipError_t hipFreeAsync(void *p, hipStream_t) { return hipFree(p); }
inline hipError_t hipMallocFromPoolAsync(void *p, size_t n, hipMemPool_t, hipStream_t) { return hipMalloc(p, n); }
inline hipError_t hipMemcpy(void *d, const void *s, size_t n, int) { memcpy(d, s, n); return hipSuccess; }
inline hipError_t hipFuncSetAttribute(const void *, int, int) { return hipSuccess; }
inline hipError_t hipDeviceGetAttribute(int *v, int a, int)
{
    *v = a == hipDeviceAttributeMultiprocessorCount ? lanes::cus : lanes::max_lds;
    return hipSuccess;
}
#define hipLaunchKernelGGL(kernel, grid, block, lds, stream, ...) \
    lanes::launch(grid, block, lds, [=]() { (void)stream; kernel(__VA_ARGS__); })
