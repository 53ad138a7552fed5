// Sums and maxima over the 64 lanes of a wave, the same in every lane.
#pragma once
#include <hip/hip_runtime.h>

namespace tmps {

// A value combined with that of the lane 32, 16, 8, 4, 2 and 1 away, each step by an instruction of the vector unit: as __shfl_xor every step is a
// way through LDS and back (some 130 cycles; a sum 0.3 us of the 3 to 4 that a normalisation or loss of a thousand rows takes).  The order of the steps makes
// a rotation by 8, 4, .. within 16 lanes what the exchange is, so that results are those of the exchanges, bit for bit.
template <class F> __device__ __forceinline__ float wave_combine(float v, F&& f) {
    {
        const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = f(__uint_as_float(s[0]), __uint_as_float(s[1]));
    }
    {
        const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = f(__uint_as_float(s[0]), __uint_as_float(s[1]));
    }
    v = f(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xF, 0xF, false)));   // row_ror:8
    v = f(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x124, 0xF, 0xF, false)));   // row_ror:4
    v = f(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x122, 0xF, 0xF, false)));   // row_ror:2
    v = f(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x121, 0xF, 0xF, false)));   // row_ror:1
    return v;
}
__device__ __forceinline__ float wsum(float v) {
    return wave_combine(v, [](float a, float b) { return a + b; });
}
__device__ __forceinline__ float wmax(float v) {
    return wave_combine(v, [](float a, float b) { return fmaxf(a, b); });
}

}  // namespace tmps
