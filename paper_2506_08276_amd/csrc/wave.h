// Wave-wide (64 lanes) sums, inner products and ordered keys of the queue kernels.
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

// One anchor row against other rows, fp32.  NV = 4-byte pieces per lane (lane l owns elements l, l + 64, ...), 0: rows
// longer than 1024, read from memory each time.  Every lane gets the result; its bits do not depend on how many rows are
// taken at once.
template <int NV>
struct RowDots {
    float a[NV > 0 ? NV : 1];
    const float *row;
    int d, lane;

    __device__ static inline float piece(__amdgpu_buffer_rsrc_t r, int lane, int j)  // 0 beyond the row's end
    {
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (j * 64 + lane) * 4, 0, 0));
    }
    __device__ inline __amdgpu_buffer_rsrc_t rsrc(const float *p) const
    {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p), 0, d * (int)sizeof(float), 0x00020000);
    }
    __device__ inline void load(const float *p, int d_, int lane_)
    {
        row = p;
        d = d_;
        lane = lane_;
        if constexpr (NV > 0) {
            const auto r = rsrc(p);
#pragma unroll
            for (int j = 0; j < NV; ++j) a[j] = piece(r, lane, j);
        }
    }
    __device__ static inline const float *uniform(const float *p)  // the same in all lanes: scalar registers
    {
        const uint64_t u = (uint64_t)p;
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u), hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
        return (const float *)((uint64_t)hi << 32 | lo);
    }
    // out[k] = <anchor, row_at(k)> for k < c <= 4.  A row's NV loads are in flight together.  The rows are not, or two by
    // two at most: both loops below test k < c, and the compiled code joins each row's loads with its sum.
    template <class RowAt>
    __device__ inline void four(RowAt row_at, int c, float (&out)[4]) const
    {
        if constexpr (NV > 0) {
            float r[4][NV];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (k < c) {
                    const auto rs = rsrc(uniform(row_at(k)));
#pragma unroll
                    for (int j = 0; j < NV; ++j) r[k][j] = piece(rs, lane, j);
                }
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (k < c) {
                    float acc = 0.f;
#pragma unroll
                    for (int j = 0; j < NV; ++j) acc = fmaf(a[j], r[k][j], acc);
                    out[k] = wave_sum(acc);
                }
        } else {
            for (int k = 0; k < c; ++k) {
                const float *e = uniform(row_at(k));
                float acc = 0.f;
                for (int i = lane; i < d; i += 64) acc = fmaf(row[i], e[i], acc);
                out[k] = wave_sum(acc);
            }
        }
    }
};

}  // namespace
