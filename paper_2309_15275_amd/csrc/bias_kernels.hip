// Column sum of g_y over all tokens: the bias gradient of a linear layer.
//
// A pass over g_y of its own would cost as much as the projection that reads the same tensor (torch's reduction:
// 30-34 us at 12608 tokens x 3072 bf16 channels, 77 MB).  The projection kernels have every patch's tokens in
// registers, and the sum of a patch is its coefficient 0 before rounding: they leave it in fp32, one row per patch
// (p^2 / 2 times fewer bytes than g_y in bf16), and column_sum_final_kernel adds those rows and the tokens outside
// the grid.  Where the projection is the generic kernel, column_sum_partial_kernel makes such rows from g_y itself.
#include "device_utils.h"
#include "kernels.h"
#include "launch.h"

namespace lbp {
namespace {

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

// rows[blockIdx.y][c] = sum of `per` tokens of gy [tokens][C]; lane = 4 channels
template <bool BF16>
__global__ __launch_bounds__(256) void column_sum_partial_kernel(const void *__restrict__ gy, long tokens, int C4, long per,
                                                                 float4 *__restrict__ rows)
{
    const int c = blockIdx.x * 256 + threadIdx.x;
    if (c >= C4) return;
    const long t0 = (long)blockIdx.y * per, t1 = min(tokens, t0 + per);
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    for (long t = t0; t < t1; ++t) add4(s, load4(gy, (size_t)t * C4 + c, BF16));
    rows[(size_t)blockIdx.y * C4 + c] = s;
}

// One workgroup: 16 channels, 256 rows at a time (4 lanes x 4 channels each), fixed order.
constexpr int kRows = 256;
template <bool BF16>
__global__ __launch_bounds__(4 * kRows) void column_sum_final_kernel(const float4 *__restrict__ rows, long Q, int C4,
                                                                     const void *__restrict__ gy, long outside, int extra,
                                                                     long img_tokens, void *__restrict__ out)
{
    __shared__ float4 red[kRows][4];
    const int g = threadIdx.x >> 2, c = blockIdx.x * 4 + (threadIdx.x & 3);
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    if (c < C4) {
        long q = g;
        for (; q + 3 * kRows < Q; q += 4 * kRows) {
            const float4 a = rows[(size_t)q * C4 + c], b = rows[(size_t)(q + kRows) * C4 + c];
            const float4 d = rows[(size_t)(q + 2 * kRows) * C4 + c], e = rows[(size_t)(q + 3 * kRows) * C4 + c];
            add4(s, a); add4(s, b); add4(s, d); add4(s, e);
        }
        for (; q < Q; q += kRows) add4(s, rows[(size_t)q * C4 + c]);
        for (long j = g; j < outside; j += kRows) {
            const long n = j / extra;
            add4(s, load4(gy, (size_t)(n * img_tokens + (j - n * extra)) * C4 + c, BF16));
        }
    }
    red[g][threadIdx.x & 3] = s;
    __syncthreads();
    for (int h = kRows / 2; h > 0; h >>= 1) {
        if (g < h) add4(red[g][threadIdx.x & 3], red[g + h][threadIdx.x & 3]);
        __syncthreads();
    }
    if (g == 0 && c < C4) {
        s = red[0][threadIdx.x];
        if (BF16) reinterpret_cast<uint2 *>(out)[c] = make_uint2(pack_bf16x2(s.x, s.y), pack_bf16x2(s.z, s.w));
        else reinterpret_cast<float4 *>(out)[c] = s;
    }
}

}  // namespace

hipError_t launch_column_sum_rows(const void *gy, long tokens, int C, int dtype, long rows, float *out, hipStream_t stream)
{
    if (tokens < 1 || C % 4 || rows < 1 || rows > 65535) return hipErrorInvalidValue;
    const int C4 = C / 4;
    const long per = (tokens + rows - 1) / rows;
    const dim3 grid((unsigned)((C4 + 255) / 256), (unsigned)rows);
    if (dtype == LBP_BF16)
        hipLaunchKernelGGL(column_sum_partial_kernel<true>, grid, dim3(256), 0, stream, gy, tokens, C4, per, (float4 *)out);
    else
        hipLaunchKernelGGL(column_sum_partial_kernel<false>, grid, dim3(256), 0, stream, gy, tokens, C4, per, (float4 *)out);
    return hipGetLastError();
}

hipError_t launch_column_sum(const float *rows, long Q, int C, const void *gy, int N, int extra, long img_tokens, int dtype,
                             void *out, hipStream_t stream)
{
    if (C % 4 || Q < 0 || extra < 0) return hipErrorInvalidValue;
    const int C4 = C / 4;
    const dim3 grid((unsigned)((C4 + 3) / 4));
    const int ex = extra > 0 ? extra : 1;
    if (dtype == LBP_BF16)
        return LBP_LAUNCH_KERNEL(column_sum_final_kernel<true>, grid, 4 * kRows, 0, stream, (const float4 *)rows, Q, C4, gy,
                                 (long)N * extra, ex, img_tokens, out);
    return LBP_LAUNCH_KERNEL(column_sum_final_kernel<false>, grid, 4 * kRows, 0, stream, (const float4 *)rows, Q, C4, gy,
                             (long)N * extra, ex, img_tokens, out);
}

}  // namespace lbp
