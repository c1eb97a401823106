// What kernels of one wavefront per column strip share: the exchange with neighbour lanes
// (DPP wave shifts; the end lanes receive 0) and buffer accesses by 32-bit byte offsets.
#pragma once
#include "internal.h"

namespace lbm {

template <int CTRL>
__device__ __forceinline__ double pair_dpp(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffLL), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
template <int CTRL>
__device__ __forceinline__ float pair_dpp(float v)
{
    return __int_as_float(
        __builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <typename T>
__device__ __forceinline__ T pair_shr(T v) { return pair_dpp<0x138>(v); }  // from lane l - 1
template <typename T>
__device__ __forceinline__ T pair_shl(T v) { return pair_dpp<0x130>(v); }  // from lane l + 1

// An offset that the hardware drops (buffers below 2 GiB), so that lanes or rows without
// an output need no branch around a store.
constexpr unsigned kPairDrop = 0x80000000u;
__device__ __forceinline__ void pair_store(__amdgpu_buffer_rsrc_t r, unsigned off, unsigned plane,
                                           double v)
{
    __builtin_amdgcn_raw_buffer_store_b64(
        __builtin_bit_cast(__attribute__((ext_vector_type(2))) int, v), r, off, plane, 0);
}
__device__ __forceinline__ void pair_store(__amdgpu_buffer_rsrc_t r, unsigned off, unsigned plane,
                                           float v)
{
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(v), r, off, plane, 0);
}
// Element at byte `off` of the plane at byte `plane` of a buffer.
__device__ __forceinline__ void pair_load(__amdgpu_buffer_rsrc_t r, unsigned off, unsigned plane,
                                          double &v)
{
    v = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, off, plane, 0));
}
__device__ __forceinline__ void pair_load(__amdgpu_buffer_rsrc_t r, unsigned off, unsigned plane,
                                          float &v)
{
    v = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, plane, 0));
}

} // namespace lbm
