// lane_ops.hpp -- compile-time loops and lane exchanges shared by the kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

namespace polarhip {

template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, E>(f);
    }
}

// Lane exchanges, all in VALU (no LDS round trip, which the early-stop test
// of the BP kernel would otherwise wait on in every iteration):
// lane ^ 1, ^ 2 by quad permutes; a lane of the other quad of its eight, the
// other half of its row of sixteen by the half-row and row mirrors (for a
// reduction any lane of the other half serves); lane ^ 16, ^ 32 by the gfx950
// row swaps.
// lane permutation CTRL of v (a full permutation of each row: every lane is
// written); the zero "old" value lets the compiler fold the move into the XOR
// that takes it
template <int CTRL>
__device__ __forceinline__ uint32_t dpp32(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false);
}

// XOR of s over each group of TL consecutive lanes (TL a power of two <= 64);
// every lane of the group gets it
template <int TL>
__device__ __forceinline__ uint32_t group_xor(uint32_t s) {
    if constexpr (TL > 1) s ^= dpp32<0xB1>(s);   // quad_perm [1,0,3,2]
    if constexpr (TL > 2) s ^= dpp32<0x4E>(s);   // quad_perm [2,3,0,1]
    if constexpr (TL > 4) s ^= dpp32<0x141>(s);  // row_half_mirror
    if constexpr (TL > 8) s ^= dpp32<0x140>(s);  // row_mirror
    if constexpr (TL > 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(s, s, false, false);
        s = r[0] ^ r[1];
    }
    if constexpr (TL > 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(s, s, false, false);
        s = r[0] ^ r[1];
    }
    return s;
}

// the value of lane + Q (Q a power of two <= 32) for the lanes whose bit Q is
// clear; what the other lanes get is not used.  Row shifts inside a row of
// sixteen; for 16 and 32 the row swaps, whose second result holds, on those
// lanes, the partner row
template <int Q>
__device__ __forceinline__ uint32_t from_lane_above(uint32_t v) {
    if constexpr (Q < 16) {
        // row_shl: lane i reads lane i + Q of its row (lanes past the row's end get 0)
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x100 + Q, 0xF, 0xF, false);
    } else if constexpr (Q == 16) {
        return __builtin_amdgcn_permlane16_swap(v, v, false, false)[1];
    } else {
        static_assert(Q == 32, "distance");
        return __builtin_amdgcn_permlane32_swap(v, v, false, false)[1];
    }
}

// orders a wavefront's own LDS accesses (other lanes' writes before the reads
// that follow)
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace polarhip
