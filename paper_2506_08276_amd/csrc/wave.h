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
constexpr int DPP_ROW_ROR8 = 0x128, DPP_ROW_ROR4 = 0x124, DPP_ROW_ROR2 = 0x122, DPP_QUAD_XOR1 = 0xB1, DPP_QUAD_XOR2 = 0x4E;

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

// Lane l's key, l the same in all lanes.
__device__ inline uint64_t key_of_lane(uint64_t k, int l)
{
    return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(k >> 32), l) << 32 | (uint32_t)__builtin_amdgcn_readlane((int)k, l);
}

// Key of lane l, another l in every lane.
__device__ inline uint64_t shfl_key(uint64_t k, int l)
{
    return (uint64_t)(uint32_t)__builtin_amdgcn_ds_bpermute(l << 2, (int)(k >> 32)) << 32 |
           (uint32_t)__builtin_amdgcn_ds_bpermute(l << 2, (int)k);
}

// The lane with the largest key (the first one of equals).
__device__ inline int wave_max_lane(uint64_t k)
{
    const uint32_t hi = (uint32_t)(k >> 32);
    unsigned long long at = __ballot(hi == wave_max(hi));
    if (__builtin_expect((at & (at - 1)) != 0, 0)) {
        const uint32_t low = hi == wave_max(hi) ? (uint32_t)k : 0u;
        at &= __ballot(low == wave_max(low));
    }
    return __ffsll((long long)at) - 1;
}

// Largest key over the wave, in every lane (0 where no lane has one).
__device__ inline uint64_t wave_max_key(uint64_t k) { return key_of_lane(k, wave_max_lane(k)); }

// Keys of LDS list `key` that are larger than k; the list is padded with zeros to a multiple of 8 entries (no key is 0).
// Eight at a time: one by one, each would wait for its own read.
__device__ inline int keys_above(const uint64_t *key, int cnt, uint64_t k)
{
    int above = 0;
    for (int j = 0; j < cnt; j += 8) {
        uint64_t v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = key[j + i];
#pragma unroll
        for (int i = 0; i < 8; ++i) above += v[i] > k;
    }
    return above;
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
    // C rows, their C * NV loads in flight together, then their sums side by side.
    template <int C, class RowAt>
    __device__ inline void rows(RowAt row_at, float (&out)[4]) const
    {
        float r[C][NV];
#pragma unroll
        for (int k = 0; k < C; ++k) {
            const auto rs = rsrc(uniform(row_at(k)));
#pragma unroll
            for (int j = 0; j < NV; ++j) r[k][j] = piece(rs, lane, j);
        }
        float acc[C];
#pragma unroll
        for (int k = 0; k < C; ++k) {
            acc[k] = 0.f;
#pragma unroll
            for (int j = 0; j < NV; ++j) acc[k] = fmaf(a[j], r[k][j], acc[k]);
        }
#pragma unroll
        for (int k = 0; k < C; ++k) out[k] = wave_sum(acc[k]);
    }
    // out[k] = <anchor, row_at(k)> for k < c, 1 <= c <= 4, c the same in all lanes.  What bounds it is one row's latency from beyond L2, so
    // the count is settled once, outside: with a test per row the compiled code waits for each row before it asks for the next.
    template <class RowAt>
    __device__ inline void four(RowAt row_at, int c, float (&out)[4]) const
    {
        if constexpr (NV > 0) {
            c = __builtin_amdgcn_readfirstlane(c);
            if (c == 1) rows<1>(row_at, out);
            else if (c == 2) rows<2>(row_at, out);
            else if (c == 3) rows<3>(row_at, out);
            else rows<4>(row_at, out);
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
