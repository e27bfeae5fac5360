// Sums over the 64 lanes of a wave in a fixed order, for the row-group kernels
// of small n.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace nbody {

// v plus v of the lane that DPP control CTRL names (all 64 lanes active).
template <int CTRL>
__device__ __forceinline__ double dpp_swap_add(double v)
{
    const auto b = __builtin_bit_cast(uint64_t, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, false);
    return v + __builtin_bit_cast(double, (uint64_t)(uint32_t)hi << 32 | (uint32_t)lo);
}

// The other half of a pair of registers: lanes 32..63 of a and lanes 0..31 of
// b change places (v_permlane32_swap_b32), then rows 1, 3 of a and rows 0, 2
// of b (v_permlane16_swap_b32; a row is 16 lanes).
__device__ __forceinline__ float swap32_add(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, a),
                                                    __builtin_bit_cast(unsigned, b), false, false);
    return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
}

__device__ __forceinline__ float swap16_add(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, a),
                                                    __builtin_bit_cast(unsigned, b), false, false);
    return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
}

// The four values of a lane in one, over four lanes each: row g of 16 lanes holds
// sums of v[quad_of_row(g)].  The four share two halvings.
__device__ __forceinline__ float quad_sums(const float (&v)[4])
{
    return swap16_add(swap32_add(v[0], v[1]), swap32_add(v[2], v[3]));
}

// Sums of R rows of four values over the 64 lanes, in a fixed order; put(k, s) is
// called with row k's total of v[k][quad_of_row(lane / 16)] in the first lane of
// every 16, for row k + 1 of a pair in the ninth.  (Every step adds lane pairs
// that exchange values, and a + b rounds as b + a: the lanes agree.)  Call with all
// 64 lanes active.
//
// Two rows share the third halving.  From the sums of four lanes (of a pair: of
// eight) on they are added in float64: a sum whose terms have one sign loses as
// much to the roundings of the last few float32 levels as to its one rounding at
// the end (p at 10,000 bodies, 2-norm: 4.2e-8 all in float32, 2.6e-8 so).
template <int R, class Put>
__device__ __forceinline__ void wave_sums(const float (&v)[R][4], int lane, Put put)
{
#pragma unroll
    for (int k = 0; k + 1 < R; k += 2) {
        const float a = quad_sums(v[k]), b = quad_sums(v[k + 1]);
        const bool second = (lane & 8) != 0;
        const float give = second ? a : b;
        const int o = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, give), 0x128, 0xF, 0xF,
                                                  false);  // row_ror:8: the other half of 16 lanes
        double s = (double)((second ? b : a) + __builtin_bit_cast(float, o));
        s = dpp_swap_add<0xB1>(s);   // quad_perm [1,0,3,2]: lane l ^ 1
        s = dpp_swap_add<0x4E>(s);   // quad_perm [2,3,0,1]: lane l ^ 2
        s = dpp_swap_add<0x141>(s);  // row_half_mirror: the other quad of 8 lanes
        if ((lane & 7) == 0) put(k + (second ? 1 : 0), s);
    }
    if constexpr (R & 1) {
        double s = (double)quad_sums(v[R - 1]);
        s = dpp_swap_add<0xB1>(s);
        s = dpp_swap_add<0x4E>(s);
        s = dpp_swap_add<0x141>(s);
        s = dpp_swap_add<0x140>(s);  // row_mirror: the other half of 16 lanes
        if ((lane & 15) == 0) put(R - 1, s);
    }
}

// Which of the four values row g (lane / 16) of quad_sums holds: 0, 2, 1, 3.
__device__ __forceinline__ int quad_of_row(int g) { return ((g & 1) << 1) | (g >> 1); }

}  // namespace nbody
