// A row of LayerNorm in the registers of 16, 32 or 64 lanes.
#pragma once

#include "common.h"
#include "gemm_common.h"

namespace sa {

template <int CTRL>
__device__ inline float dpp_add(float v) {
    const int other = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true);
    return v + __builtin_bit_cast(float, other);
}

// Sum over aligned groups of LPR lanes (16, 32 or 64) as a butterfly, the most distant lanes first; every lane of a group
// gets it.  Once lanes 8 apart agree, a rotation of the 16 lanes of a row by 4 (then 2, 1) is an exchange of neighbours.
template <int LPR>
__device__ inline float group_sum(float v) {
    if (LPR == 64) {
        const uint32_t u = __builtin_bit_cast(uint32_t, v);
        const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
        const uint32_t r0 = r[0], r1 = r[1];
        v = __builtin_bit_cast(float, r0) + __builtin_bit_cast(float, r1);
    }
    if (LPR >= 32) {
        const uint32_t u = __builtin_bit_cast(uint32_t, v);
        const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
        const uint32_t r0 = r[0], r1 = r[1];
        v = __builtin_bit_cast(float, r0) + __builtin_bit_cast(float, r1);
    }
    v = dpp_add<0x128>(v);                // row_ror:8
    v = dpp_add<0x124>(v);                // row_ror:4
    v = dpp_add<0x122>(v);                // row_ror:2
    v = dpp_add<0x121>(v);                // row_ror:1
    return v;
}

// A lane's part of a row, zero in the lanes past the row's end.  Those load the row's end like the last lane inside: a choice between
// an address in memory and a constant made the compiler put the constant on the stack and load through both (E = 192: flat loads,
// and a wait for every load under way, the weights' among them; layer of 12608 x 192, 768 hidden 68.3 -> 66.7 us without).
__device__ inline float4 row_or_zero(const float4 &v, bool in) {
    return make_float4(in ? v.x : 0.0f, in ? v.y : 0.0f, in ? v.z : 0.0f, in ? v.w : 0.0f);
}

// Of a row of E elements, lane l's at 4 (c LPR + l): mean, and 1 / sqrt(variance + eps).
template <int LPR, int CH>
__device__ inline void row_stats(const float4 (&v)[CH], int l, int E, float eps, float &mean, float &rstd) {
    float s = 0.0f;
#pragma unroll
    for (int c = 0; c < CH; ++c) s += (v[c].x + v[c].y) + (v[c].z + v[c].w);
    mean = group_sum<LPR>(s) / (float)E;
    float ss = 0.0f;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const int j = (c * LPR + l) * 4;
        if (j < E) {
            const float d0 = v[c].x - mean, d1 = v[c].y - mean, d2 = v[c].z - mean, d3 = v[c].w - mean;
            ss += (d0 * d0 + d1 * d1) + (d2 * d2 + d3 * d3);
        }
    }
    rstd = 1.0f / __builtin_sqrtf(group_sum<LPR>(ss) / (float)E + eps);
}

__device__ inline void normalise(const float4 &v, float mean, float rstd, const float4 &g, const float4 &b, float (&y)[4]) {
    y[0] = (v.x - mean) * rstd * g.x + b.x;
    y[1] = (v.y - mean) * rstd * g.y + b.y;
    y[2] = (v.z - mean) * rstd * g.z + b.z;
    y[3] = (v.w - mean) * rstd * g.w + b.w;
}

__device__ inline uint32_t codes_of(const float (&y)[4], float inv_scale) {
    return requant_bytes(y[0] * inv_scale, y[1] * inv_scale, y[2] * inv_scale, y[3] * inv_scale);
}

}  // namespace sa
