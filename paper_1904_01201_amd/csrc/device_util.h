// Wave and block helpers and triangle loads shared by the kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dtypes.h"
#include "raster_math.h"

#pragma clang fp contract(off)

namespace habmi {

// ------------------------------------------------------------ wave helpers
__device__ __forceinline__ uint32_t lane_id() { return __lane_id(); }

// A value every lane of the wave holds alike, moved to a scalar register so
// that what it indexes is fetched through the scalar cache.
__device__ __forceinline__ uint32_t uniform(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }

__device__ __forceinline__ unsigned long long lanemask_lt()
{
    return (1ull << lane_id()) - 1ull;
}

__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t x)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
    return x;
}

// Exclusive scan over the block (NT threads, wave64); *total gets the sum.
// wtot: LDS scratch of NT/64 words.  Contains two barriers.
template <int NT>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t x, uint32_t *wtot, uint32_t *total)
{
    const uint32_t lane = lane_id(), wave = threadIdx.x >> 6;
    uint32_t s = x;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        uint32_t y = __shfl_up(s, off);
        if (lane >= (uint32_t)off) s += y;
    }
    if (lane == 63) wtot[wave] = s;
    __syncthreads();
    uint32_t pre = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) {
        uint32_t v = wtot[w];
        pre += (w < (int)wave) ? v : 0u;
        tot += v;
    }
    __syncthreads();
    *total = tot;
    return pre + s - x;
}

__device__ __forceinline__ uint2 pack_box(const PixBox &b)
{
    return make_uint2((uint32_t)b.i0 | ((uint32_t)b.j0 << 16), (uint32_t)b.i1 | ((uint32_t)b.j1 << 16));
}

// A pointer read out of a view record, known to point into device global
// memory: loads through it are global (vector memory only), not flat.
template <typename T>
__device__ __forceinline__ const __attribute__((address_space(1))) T *gmem(const T *p)
{
    return (const __attribute__((address_space(1))) T *)p;
}
template <typename T>
__device__ __forceinline__ __attribute__((address_space(1))) T *gmem_out(T *p)
{
    return (__attribute__((address_space(1))) T *)p;
}

// Triangle t's vertex positions: nine consecutive floats of the
// per-triangle copy, independent loads (no dependent index -> position
// load).  With T up to 2^30, 9 t can exceed 32 bits: a 64-bit offset.
__device__ __forceinline__ void load_pos(const DView &v, uint32_t t, float P[9])
{
    const auto *p = gmem(v.tpos) + 9ull * t;
#pragma unroll
    for (int i = 0; i < 9; ++i) P[i] = p[i];
}

}  // namespace habmi
