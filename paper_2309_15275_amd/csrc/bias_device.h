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

// Chains of rows that are added up side by side, row by row, and then two by two, whoever adds them: a workgroup of fewer threads gives a lane
// several, so that the order of the sum, hence its bits, is that of the kernel of its own.  (A chain for each row of threads was a
// sum of chains two to four times as long: 25088 rows on 64 x 64 tiles, fp32 error 3.7e-7 against 1.9e-7.)
// What bounds it is the chain of reads.  Beside the products it is faster than in a kernel of its own for any number of rows, as most of it
// runs while those do.  Whole backward calls, own kernel / beside (us): 32 rows 48 -> 192 channels 13.0 / 10.5, 256 rows 768 -> 3072
// 52.0 / 47.7, 6272 rows 384 -> 384 146 / 134, 25088 rows (4 x 4 patches) 48 -> 192 99.5 / 87.0, 128 -> 512 198 / 185; of 170 layers of 32 to
// 25088 rows none is slower.
constexpr int kBiasRows = 256;

// One workgroup of 4 * ROWS threads: 16 channels, 4 lanes x 4 channels a row, CHAINS of the chains a lane.  red: 4 * ROWS values of LDS.
template <int ROWS, bool BF16>
__device__ __forceinline__ void bias_sum_block(const BiasSum &b, int block, float4 *red)
{
    constexpr int CHAINS = kBiasRows / ROWS, ROUNDS = CHAINS > 2 ? 2 : 4;      // reads in flight: 4 or 8
    const int g = threadIdx.x >> 2, l = threadIdx.x & 3, c = block * 4 + l;
    const size_t C4 = b.C4;
    float4 s[CHAINS];
#pragma unroll
    for (int v = 0; v < CHAINS; ++v) s[v] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (c < b.C4) {
        long q = g;
        for (; q + (CHAINS - 1) * ROWS + (ROUNDS - 1) * kBiasRows < b.Q; q += ROUNDS * kBiasRows) {
            float4 row[ROUNDS][CHAINS];
#pragma unroll
            for (int u = 0; u < ROUNDS; ++u)
#pragma unroll
                for (int v = 0; v < CHAINS; ++v) row[u][v] = b.rows[(size_t)(q + u * kBiasRows + v * ROWS) * C4 + c];
#pragma unroll
            for (int u = 0; u < ROUNDS; ++u)
#pragma unroll
                for (int v = 0; v < CHAINS; ++v) add4(s[v], row[u][v]);
        }
        for (; q < b.Q; q += kBiasRows) {
            float4 row[CHAINS];
#pragma unroll
            for (int v = 0; v < CHAINS; ++v) row[v] = b.rows[(size_t)min(q + v * ROWS, (long)b.Q - 1) * C4 + c];
#pragma unroll
            for (int v = 0; v < CHAINS; ++v)
                if (q + v * ROWS < b.Q) add4(s[v], row[v]);
        }
        for (int j = g; j < b.outside; j += kBiasRows) {
            float4 row[CHAINS];
#pragma unroll
            for (int v = 0; v < CHAINS; ++v) {
                const int i = min(j + v * ROWS, b.outside - 1), n = i / b.extra;
                row[v] = load4(b.gy, ((size_t)n * b.img_tokens + (i - n * b.extra)) * C4 + c, BF16);
            }
#pragma unroll
            for (int v = 0; v < CHAINS; ++v)
                if (j + v * ROWS < b.outside) add4(s[v], row[v]);
        }
    }
#pragma unroll
    for (int h = CHAINS / 2; h > 0; h >>= 1)
#pragma unroll
        for (int v = 0; v < h; ++v) add4(s[v], s[v + h]);
    red[g * 4 + l] = s[0];
    __syncthreads();
    for (int h = ROWS / 2; h > 0; h >>= 1) {
        if (g < h) add4(red[g * 4 + l], red[(g + h) * 4 + l]);
        __syncthreads();
    }
    if (g == 0 && c < b.C4) {
        const float4 sum = red[l];
        if (BF16) reinterpret_cast<uint2 *>(b.out)[c] = make_uint2(pack_bf16x2(sum.x, sum.y), pack_bf16x2(sum.z, sum.w));
        else reinterpret_cast<float4 *>(b.out)[c] = sum;
    }
}

}  // namespace lbp
