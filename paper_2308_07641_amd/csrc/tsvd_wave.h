// Sums over a wavefront in fp64, for the kernels of the transition.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace {

// The value of lane ^ J of the wavefront, by cross-lane moves of the vector ALU (about ten cycles; a shuffle through
// the LDS crossbar takes over a hundred).
template <int J>
__device__ __forceinline__ uint32_t lane_xor32(uint32_t x) {
    if constexpr (J == 1) return __builtin_amdgcn_mov_dpp(x, 0xB1, 0xF, 0xF, true);            // quad_perm 1,0,3,2
    else if constexpr (J == 2) return __builtin_amdgcn_mov_dpp(x, 0x4E, 0xF, 0xF, true);       // quad_perm 2,3,0,1
    else if constexpr (J == 4) return __builtin_amdgcn_mov_dpp(__builtin_amdgcn_mov_dpp(x, 0x141, 0xF, 0xF, true), 0x1B, 0xF, 0xF, true);   // ^ 7, ^ 3
    else if constexpr (J == 8) return __builtin_amdgcn_mov_dpp(x, 0x128, 0xF, 0xF, true);      // row_ror 8
    else if constexpr (J == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        return (threadIdx.x & 16) ? r[0] : r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        return (threadIdx.x & 32) ? r[0] : r[1];
    }
}
template <int J>
__device__ __forceinline__ double lane_xor(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    return __builtin_bit_cast(double, (uint64_t)lane_xor32<J>((uint32_t)b) | ((uint64_t)lane_xor32<J>((uint32_t)(b >> 32)) << 32));
}

// Sum over a wavefront, in every lane.
__device__ __forceinline__ double wave_sum(double v) {
    v += lane_xor<32>(v);
    v += lane_xor<16>(v);
    v += lane_xor<8>(v);
    v += lane_xor<4>(v);
    v += lane_xor<2>(v);
    v += lane_xor<1>(v);
    return v;
}

// Sum over the lanes up to and including one's own: rows of 16 lanes, then the totals of the rows before.
template <int CTRL, int ROWS>
__device__ __forceinline__ double lane_shifted(double v) {      // zero where the move has no source
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, (uint32_t)b, CTRL, ROWS, 0xF, false), hi = __builtin_amdgcn_update_dpp(0, (uint32_t)(b >> 32), CTRL, ROWS, 0xF, false);
    return __builtin_bit_cast(double, (uint64_t)lo | ((uint64_t)hi << 32));
}
__device__ __forceinline__ double wave_scan(double v) {
    v += lane_shifted<0x111, 0xF>(v);            // row_shr 1, 2, 4, 8
    v += lane_shifted<0x112, 0xF>(v);
    v += lane_shifted<0x114, 0xF>(v);
    v += lane_shifted<0x118, 0xF>(v);
    v += lane_shifted<0x142, 0xA>(v);            // row_bcast 15 into rows 1 and 3
    v += lane_shifted<0x143, 0xC>(v);            // row_bcast 31 into rows 2 and 3
    return v;
}

}  // namespace
