// Exchanges between the lanes of a wavefront that stay out of the LDS unit.
#pragma once
#include <hip/hip_runtime.h>

// The value of lane (own ^ O), by DPP and permlane moves: a butterfly of __shfl_xor is a chain of trips through the LDS
// unit, for the sampler most of what a workgroup waits for when it sums one slice after another.
// (quad_perm 1 0 3 2 and 2 3 0 1; half-row mirror, then the quad mirrored back; a row rotated by eight; rows and halves
// swapped: the results of a swap of a register with itself are own and partner, in an order that depends on the lane)
template <int O>
__device__ __forceinline__ unsigned lane_xor(unsigned v) {
    if constexpr (O == 1) return __builtin_amdgcn_update_dpp(0u, v, 0xB1, 0xF, 0xF, true);
    else if constexpr (O == 2) return __builtin_amdgcn_update_dpp(0u, v, 0x4E, 0xF, 0xF, true);
    else if constexpr (O == 4)
        return __builtin_amdgcn_update_dpp(0u, __builtin_amdgcn_update_dpp(0u, v, 0x141, 0xF, 0xF, true), 0x1B, 0xF, 0xF, true);
    else if constexpr (O == 8) return __builtin_amdgcn_update_dpp(0u, v, 0x128, 0xF, 0xF, true);
    else {
        static_assert(O == 16 || O == 32, "within a wavefront");
        const auto sw = O == 16 ? __builtin_amdgcn_permlane16_swap(v, v, false, false) : __builtin_amdgcn_permlane32_swap(v, v, false, false);
        return (threadIdx.x & O) ? sw[0] : sw[1];
    }
}
