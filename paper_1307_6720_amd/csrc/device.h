// Device helpers shared by the kernel translation units.
#pragma once

#include <type_traits>

#include "internal.h"

namespace mhs {
namespace {

// Descriptor pointers arrive without an address space, which would make every
// access a FLAT instruction; FLAT counts against the LDS wait counter too, so
// each LDS barrier would also wait for all outstanding HBM loads.  All
// buffers are device (global) memory: say so.
#define MHS_GLOBAL __attribute__((address_space(1)))
template <typename T>
__device__ __forceinline__ const MHS_GLOBAL T *gin(const void *p)
{
    return (const MHS_GLOBAL T *)p;
}
template <typename T>
__device__ __forceinline__ MHS_GLOBAL T *gout(void *p)
{
    return (MHS_GLOBAL T *)p;
}
// Small read-only tables indexed by workgroup-uniform values (per-plane
// coefficients): the constant address space lets them use scalar loads,
// which do not share the vector-memory wait counter with the plane prefetch.
#define MHS_CONST __attribute__((address_space(4)))
template <typename T>
__device__ __forceinline__ const MHS_CONST T *gconst(const void *p)
{
    return (const MHS_CONST T *)p;
}

// One plane of an array as a buffer resource (base address and byte length
// in scalar registers): loads and stores then take a 32-bit per-lane byte
// offset with no 64-bit address arithmetic per access, and an offset at or
// past the length reads zero.  Word 3 selects raw 32-bit dword access.
constexpr int kBufWord3 = 0x00020000;
template <typename T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(const MHS_GLOBAL T *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc((void *)base, (short)0, (int)bytes, kBufWord3);
}
template <typename T>
__device__ __forceinline__ T bload(__amdgpu_buffer_rsrc_t r, uint32_t off);
template <>
__device__ __forceinline__ float bload<float>(__amdgpu_buffer_rsrc_t r, uint32_t off)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}
template <>
__device__ __forceinline__ double bload<double>(__amdgpu_buffer_rsrc_t r, uint32_t off)
{
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}
__device__ __forceinline__ void bstore(float v, __amdgpu_buffer_rsrc_t r, uint32_t off)
{
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, off, 0, 0);
}
__device__ __forceinline__ void bstore(double v, __amdgpu_buffer_rsrc_t r, uint32_t off)
{
    typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, off, 0, 0);
}
template <typename Item>
__device__ __forceinline__ int find_item(const Item *items, int n, int tile)
{
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (items[mid].tile_base <= tile)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// Workgroup barrier that orders LDS traffic only.  The kernels share data
// between threads exclusively through LDS, so the barrier must not wait for
// outstanding global loads (a plain __syncthreads() would, which drains the
// prefetch ring at every step) or stores.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Workgroups are dispatched round-robin over the 8 XCDs (block b runs on XCD
// b % 8), each with its own L2.  Remap so that each XCD receives one
// contiguous range of tiles: neighbouring tiles, which re-read each other's
// halo rows, then share an L2 and run at about the same time.
constexpr int kXcds = 8;
__device__ __forceinline__ int xcd_tile()
{
    const int nb = (int)gridDim.x, b = (int)blockIdx.x;
    const int x = b % kXcds, q = b / kXcds;
    const int per = nb / kXcds, rem = nb % kXcds;
    return x * per + min(x, rem) + q;
}
// A launch whose items have different shapes (requests of several sizes
// merged by the batch) takes its tiles in dispatch order instead: its items'
// tiles march different numbers of planes, and contiguous ranges would give
// some XCDs only the long marches.
__device__ __forceinline__ int launch_tile(const LevelItem *items, int nitems)
{
    return (nitems > 1 && items[0].spread) ? (int)blockIdx.x : xcd_tile();
}

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Fixed-order block sum (deterministic); result valid in thread 0.
template <int NT>
__device__ __forceinline__ double block_sum(double v, double *red)
{
    v = wave_sum(v);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) red[w] = v;
    lds_barrier();
    double s = 0.0;
    if (threadIdx.x == 0) {
#pragma unroll
        for (int q = 0; q < NT / 64; ++q) s += red[q];
    }
    return s;
}

// Per-plane coefficients of planes base .. base+63, one plane per lane of
// every wave: the z-march reads plane p's value with a lane broadcast
// (v_readlane, the index is wave-uniform) instead of a scalar memory load
// whose wait would also hold up the LDS traffic of the step.
__device__ __forceinline__ float lane_bcast(float v, int lane)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}
__device__ __forceinline__ double lane_bcast(double v, int lane)
{
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffLL), lane);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}
template <typename T>
struct PlaneTab {
    T v;
    int base;
    __device__ __forceinline__ void load(const MHS_CONST T *coef, int b, int comp, int nz)
    {
        base = b;
        const int p = b + (int)(threadIdx.x & 63);
        v = (p >= 0 && p < nz) ? coef[4 * p + comp] : (T)0;
    }
    __device__ __forceinline__ T operator()(int p) const { return lane_bcast(v, p - base); }
};

} // namespace
} // namespace mhs
