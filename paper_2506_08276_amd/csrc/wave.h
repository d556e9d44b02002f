// Wave-wide (64 lanes) sums and ordered keys of the queue kernels.
#pragma once
#include "common.h"

namespace {

// Lane permutations inside a row of 16: rotation by n lanes, and lane ^ 1.
template <int CTRL>
__device__ inline uint32_t dpp_mov(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}
constexpr int DPP_ROW_ROR8 = 0x128, DPP_ROW_ROR4 = 0x124, DPP_ROW_ROR2 = 0x122, DPP_QUAD_XOR1 = 0xB1;

// Sum over the wave, in every lane.  The additions are those of a butterfly over lane ^ 32, 16, 8, 4, 2, 1 (after the
// step over lane ^ 8 the values repeat every 8 lanes, so a rotation by 4 reaches lane ^ 4, and so on), so the bits are the
// butterfly's; the lane exchanges are register moves instead of trips through the LDS crossbar.
__device__ inline float wave_sum(float v)
{
    {
        const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = __uint_as_float(p[0]) + __uint_as_float(p[1]);
    }
    {
        const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = __uint_as_float(p[0]) + __uint_as_float(p[1]);
    }
    v += __uint_as_float(dpp_mov<DPP_ROW_ROR8>(__float_as_uint(v)));
    v += __uint_as_float(dpp_mov<DPP_ROW_ROR4>(__float_as_uint(v)));
    v += __uint_as_float(dpp_mov<DPP_ROW_ROR2>(__float_as_uint(v)));
    v += __uint_as_float(dpp_mov<DPP_QUAD_XOR1>(__float_as_uint(v)));
    return v;
}

// Largest value over the wave, in every lane.
__device__ inline uint32_t wave_max(uint32_t v)
{
    {
        const auto p = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        v = p[0] > p[1] ? p[0] : p[1];
    }
    {
        const auto p = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        v = p[0] > p[1] ? p[0] : p[1];
    }
    uint32_t w = dpp_mov<DPP_ROW_ROR8>(v);
    v = v > w ? v : w;
    w = dpp_mov<DPP_ROW_ROR4>(v);
    v = v > w ? v : w;
    w = dpp_mov<DPP_ROW_ROR2>(v);
    v = v > w ? v : w;
    w = dpp_mov<DPP_QUAD_XOR1>(v);
    return v > w ? v : w;
}

// (score, id) as one integer whose order is "score descending, id ascending": the larger key is the better entry.  Both
// zeros are one score, NaN ranks below everything.  No key is 0.
__device__ inline uint32_t score_bits(float s)
{
    const uint32_t u = __float_as_uint(s + 0.0f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return 0u;
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ inline uint64_t queue_key(float s, uint32_t id) { return ((uint64_t)score_bits(s) << 32) | (uint32_t)~id; }
__device__ inline uint32_t key_id(uint64_t k) { return ~(uint32_t)k; }
__device__ inline float key_score(uint64_t k)
{
    const uint32_t h = (uint32_t)(k >> 32);
    return __uint_as_float((h & 0x80000000u) ? (h & 0x7fffffffu) : ~h);
}

// Largest key over the wave, in every lane (0 where no lane has one).
__device__ inline uint64_t wave_max_key(uint64_t k)
{
    const uint32_t hi = (uint32_t)(k >> 32), top = wave_max(hi);
    const uint32_t low = wave_max(hi == top ? (uint32_t)k : 0u);
    return ((uint64_t)top << 32) | low;
}

}  // namespace
