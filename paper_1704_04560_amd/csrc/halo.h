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

}  // namespace mtx
