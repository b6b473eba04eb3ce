// Wavefront-level scans and lane exchanges (64-lane wavefronts).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace p4q {

// Inclusive prefix sum over the 64 lanes of a wavefront with DPP row shifts
// and row broadcasts (no LDS round trips).
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, true);  // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, true);  // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, true);  // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, true);  // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false); // row_bcast:15
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false); // row_bcast:31
    return v;
}

// x of lane ^ M, M < 16, by DPP (4: mirrored halves of 8, mirrored quads)
template <int M>
__device__ __forceinline__ uint32_t lane_xor(uint32_t x) {
    static_assert(M == 1 || M == 2 || M == 4 || M == 8, "one bit of the lane number within a row");
    int v = (int)x;
    if constexpr (M == 8) v = __builtin_amdgcn_update_dpp(0, v, 0x128, 0xF, 0xF, true);       // row_ror:8
    if constexpr (M == 4) {
        v = __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, true);                         // row_half_mirror
        v = __builtin_amdgcn_update_dpp(0, v, 0x1B, 0xF, 0xF, true);                          // quad_perm 3,2,1,0
    }
    if constexpr (M == 2) v = __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, true);        // quad_perm 2,3,0,1
    if constexpr (M == 1) v = __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, true);        // quad_perm 1,0,3,2
    return (uint32_t)v;
}

// sum of wtot[0 .. wave) read as four 16-byte words (up to 16 wavefronts)
__device__ __forceinline__ uint32_t waves_before(const uint32_t *wtot, int wave) {
    const uint4 *w4 = reinterpret_cast<const uint4 *>(wtot);
    uint32_t s = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint4 v = w4[q];
        s += (4 * q + 0 < wave ? v.x : 0u) + (4 * q + 1 < wave ? v.y : 0u) +
             (4 * q + 2 < wave ? v.z : 0u) + (4 * q + 3 < wave ? v.w : 0u);
    }
    return s;
}

}  // namespace p4q
