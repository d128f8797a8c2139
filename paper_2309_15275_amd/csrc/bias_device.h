// The last stage of the bias gradient (bias_kernels.hip): the sum of fp32 rows and of the tokens outside the grid, for 16 channels.  A
// kernel of its own runs it, and so do workgroups at the end of a grouped launch of both products.
#pragma once
#include "device_utils.h"

namespace lbp {

struct BiasSum {
    const float4 *rows;      // [Q][C]
    const void *gy;          // tokens outside the grid: `extra` in front of every image's
    void *out;               // [C], of the tensor's type
    int Q, C4;               // rows, channels / 4
    int outside, extra;      // N * extra of them
    long img_tokens;
    int blocks;              // workgroups: 16 channels each
};

inline int bias_sum_blocks(int C) { return (C / 4 + 3) / 4; }

__device__ __forceinline__ float4 load4(const void *p, size_t i, bool bf16)
{
    if (!bf16) return reinterpret_cast<const float4 *>(p)[i];
    const uint2 u = reinterpret_cast<const uint2 *>(p)[i];
    return make_float4(bf16_lo_to_f32(u.x), bf16_hi_to_f32(u.x), bf16_lo_to_f32(u.y), bf16_hi_to_f32(u.y));
}

__device__ __forceinline__ void add4(float4 &s, const float4 &v)
{
    s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
}

// One workgroup of 4 * ROWS threads: 16 channels, ROWS rows at a time (4 lanes x 4 channels each), fixed order.  red: 4 * ROWS values of LDS.
template <int ROWS, bool BF16>
__device__ __forceinline__ void bias_sum_block(const BiasSum &b, int block, float4 *red)
{
    const int g = threadIdx.x >> 2, l = threadIdx.x & 3, c = block * 4 + l;
    const size_t C4 = b.C4;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    if (c < b.C4) {
        long q = g;
        for (; q + 3 * ROWS < b.Q; q += 4 * ROWS) {
            const float4 r0 = b.rows[(size_t)q * C4 + c], r1 = b.rows[(size_t)(q + ROWS) * C4 + c];
            const float4 r2 = b.rows[(size_t)(q + 2 * ROWS) * C4 + c], r3 = b.rows[(size_t)(q + 3 * ROWS) * C4 + c];
            add4(s, r0); add4(s, r1); add4(s, r2); add4(s, r3);
        }
        for (; q < b.Q; q += ROWS) add4(s, b.rows[(size_t)q * C4 + c]);
        for (int j = g; j < b.outside; j += ROWS) {
            const int n = j / b.extra;
            add4(s, load4(b.gy, ((size_t)n * b.img_tokens + (j - n * b.extra)) * C4 + c, BF16));
        }
    }
    red[g * 4 + l] = s;
    __syncthreads();
    for (int h = ROWS / 2; h > 0; h >>= 1) {
        if (g < h) add4(red[g * 4 + l], red[(g + h) * 4 + l]);
        __syncthreads();
    }
    if (g == 0 && c < b.C4) {
        s = red[l];
        if (BF16) reinterpret_cast<uint2 *>(b.out)[c] = make_uint2(pack_bf16x2(s.x, s.y), pack_bf16x2(s.z, s.w));
        else reinterpret_cast<float4 *>(b.out)[c] = s;
    }
}

}  // namespace lbp
