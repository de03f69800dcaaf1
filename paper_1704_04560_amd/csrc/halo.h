// Shared by the convolutions over input windows held in LDS (conv_halo.hip, conv_halo_wgrad.hip).
#pragma once

#include "igemm.h"

namespace mtx {

constexpr int kHaloMaxLds = 80 * 1024;  // two blocks per compute unit

static inline int halo_cdiv(int a, int b) { return (a + b - 1) / b; }

// Element c .. c+7 of the input at element offset off (of channel c); channels from `left` on
// are zero.  VIN = 8, 4 or 1: channels per load that alignment and the channel count allow.
template <int VIN>
__device__ __forceinline__ u32x4 halo_granule(const __amdgpu_buffer_rsrc_t r, bool ok, int off, int left)
{
    if constexpr (VIN == 8)
        return __builtin_amdgcn_raw_buffer_load_b128(r, ok && (left > 0) ? off * 2 : (int)kOOB, 0, 0);
    u32x4 v;
    if constexpr (VIN == 4) {
        const u32x2 lo = __builtin_amdgcn_raw_buffer_load_b64(r, ok && (left > 0) ? off * 2 : (int)kOOB, 0, 0);
        const u32x2 hi = __builtin_amdgcn_raw_buffer_load_b64(r, ok && (left > 4) ? off * 2 + 8 : (int)kOOB, 0, 0);
        return u32x4{lo[0], lo[1], hi[0], hi[1]};
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const unsigned a = __builtin_amdgcn_raw_buffer_load_b16(
            r, ok && (left > 2 * i) ? off * 2 + 4 * i : (int)kOOB, 0, 0);
        const unsigned b = __builtin_amdgcn_raw_buffer_load_b16(
            r, ok && (left > 2 * i + 1) ? off * 2 + 4 * i + 2 : (int)kOOB, 0, 0);
        v[i] = (a & 0xffffu) | (b << 16);
    }
    return v;
}

// Output rows in pieces of 8 channels: 16-byte accesses where a group's channels are a multiple of
// 8 (width 8), 8-byte ones where they are a multiple of 4 (width 4), else single ones (width 1, in
// the kernels).  With single ones at 396 channels, the data gradient of 1856 images of 16 x 3
// (3 x 3, from 8 channels) took 115 us, with 8-byte ones 58, the implicit GEMM 74.  `left`: channels
// of the row from this piece on.
static inline int halo_row_width(int channels) { return channels % 8 == 0 ? 8 : channels % 4 == 0 ? 4 : 1; }

// (The width is a compile-time one: a branch on it for every piece, between the loads and stores of a
// block, cost the CIFAR and AlexNet steps half a percent.)
template <int W>
__device__ __forceinline__ u32x4 halo_row_load(const __amdgpu_buffer_rsrc_t r, bool ok, int idx, int left)
{
    if constexpr (W == 8)
        return __builtin_amdgcn_raw_buffer_load_b128(r, ok && left > 0 ? idx * 2 : (int)kOOB, 0, 0);
    const u32x2 lo = __builtin_amdgcn_raw_buffer_load_b64(r, ok && left > 0 ? idx * 2 : (int)kOOB, 0, 0);
    const u32x2 hi = __builtin_amdgcn_raw_buffer_load_b64(r, ok && left > 4 ? idx * 2 + 8 : (int)kOOB, 0, 0);
    return u32x4{lo[0], lo[1], hi[0], hi[1]};
}

template <int W>
__device__ __forceinline__ void halo_row_store(bf16_t* p, u32x4 v, int left)
{
    if constexpr (W == 8) {
        *reinterpret_cast<u32x4*>(p) = v;
    } else {
        reinterpret_cast<u32x2*>(p)[0] = u32x2{v[0], v[1]};
        if (left > 4) reinterpret_cast<u32x2*>(p)[1] = u32x2{v[2], v[3]};
    }
}

// v where the mask (the stored output of a ReLU) is positive, else zero
__device__ __forceinline__ u32x4 halo_masked(u32x4 v, u32x4 m)
{
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const unsigned lo = __uint_as_float(m[e] << 16) > 0.f ? 0xffffu : 0u;
        const unsigned hi = __uint_as_float(m[e] & 0xffff0000u) > 0.f ? 0xffff0000u : 0u;
        v[e] &= lo | hi;
    }
    return v;
}

}  // namespace mtx
