// Eight dot products at a time: every lane of an aligned run of LC lanes holds its share of eight sums, and the run
// adds them up while it hands them round, so that each step halves the sums a lane carries (8, 4, 2, 1) as it doubles
// the lanes behind each.  At strides 32 and 16 one lane swap and one addition do two sums, below that row shifts under
// a bank mask and quad permutes; nothing goes through the LDS crossbar.  For LC = 64 the eight sums cost 19 vector
// instructions, for LC = 32 (two runs in the wavefront) 22, where eight separate tree sums take 48 and 40.
#pragma once
#include "sgap_common.hpp"

namespace sgap {

template <int CTRL, int BANKS>
__device__ __forceinline__ float dpp_into(float old, float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, old), __builtin_bit_cast(int, v),
                                                                 CTRL, 0xF, BANKS, false));
}

// Lanes with bit S of their number clear: the sum of a over this lane and the one S above; bit set: the sum of b over
// this lane and the one S below.
template <int S>
__device__ __forceinline__ float pair_step(float a, float b)
{
    if constexpr (S == 32) {
        auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b), false, false);
        const unsigned x = r[0], y = r[1];  // scalars first: bit_cast of a vector element misreads
        return __builtin_bit_cast(float, x) + __builtin_bit_cast(float, y);
    } else if constexpr (S == 16) {
        auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b), false, false);
        const unsigned x = r[0], y = r[1];
        return __builtin_bit_cast(float, x) + __builtin_bit_cast(float, y);
    } else if constexpr (S == 8 || S == 4) {
        constexpr int LOW = S == 8 ? 0x3 : 0x5, HIGH = S == 8 ? 0xC : 0xA;  // banks of four lanes with the bit clear / set
        const float keep = dpp_into<0xE4, HIGH>(a, b);                      // quad_perm identity: b where the bit is set
        const float came = dpp_into<0x110 + S, HIGH>(dpp_into<0x100 + S, LOW>(0.0f, a), b);  // row_shl / row_shr by S
        return keep + came;
    } else {
        static_assert(S == 2 || S == 1, "strides of a wavefront");
        const bool up = (threadIdx.x & S) != 0;
        const float keep = up ? b : a;
        const float give = up ? a : b;
        return keep + dpp_into<S == 2 ? 0x4E : 0xB1, 0xF>(0.0f, give);  // quad_perm [2,3,0,1] / [1,0,3,2]
    }
}

// One sum left: add the lane S above (valid in the lanes with bit S clear, and all below it).
template <int S>
__device__ __forceinline__ float last_steps(float v)
{
    if constexpr (S >= 1) {
        if constexpr (S >= 4) v += dpp_into<0x100 + S, 0xF>(0.0f, v);
        else v += dpp_into<S == 2 ? 0x4E : 0xB1, 0xF>(0.0f, v);
        return last_steps<S / 2>(v);
    } else {
        return v;
    }
}

template <int S, int V>
__device__ __forceinline__ void dot8_steps(float (&v)[8])
{
    if constexpr (V > 1) {
#pragma unroll
        for (int i = 0; i < V / 2; ++i) v[i] = pair_step<S>(v[i], v[i + V / 2]);
        dot8_steps<S / 2, V / 2>(v);
    } else {
        v[0] = last_steps<S>(v[0]);
    }
}

// Afterwards v[0] is complete in the lanes with dot8_writer() and belongs to the sum number dot8_number() of the eight.
// All lanes of the wavefront call together.
template <int LC>
__device__ __forceinline__ void dot8_reduce(float (&v)[8])
{
    static_assert(LC >= 8 && LC <= 64, "8 to 64 lanes");
    dot8_steps<LC / 2, 8>(v);
}
template <int LC>
__device__ __forceinline__ bool dot8_writer(int chunk) { return chunk % (LC / 8) == 0; }
template <int LC>
__device__ __forceinline__ int dot8_number(int chunk) { return chunk / (LC / 8); }

}  // namespace sgap
