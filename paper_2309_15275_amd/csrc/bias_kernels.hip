// Column sum of g_y over all tokens: the bias gradient of a linear layer.
//
// A pass over g_y of its own would cost as much as the projection that reads the same tensor (torch's reduction:
// 30-34 us at 12608 tokens x 3072 bf16 channels, 77 MB).  The projection kernels have every patch's tokens in
// registers, and the sum of a patch is its coefficient 0 before rounding: they leave it in fp32, one row per patch
// (p^2 / 2 times fewer bytes than g_y in bf16), and column_sum_final_kernel adds those rows and the tokens outside
// the grid.  Where the projection is the generic kernel, column_sum_partial_kernel makes such rows from g_y itself.
// Where both products of a call are one launch, workgroups at its end add the rows up (bias_device.h) in place of a launch between the
// projection and the products: 4.7 us and a gap of 1.5 in the step of a layer of 12608 tokens 768 -> 3072, 121 us.
#include "bias_device.h"
#include "device_utils.h"
#include "kernels.h"
#include "launch.h"

namespace lbp {
namespace {

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

template <bool BF16>
__global__ __launch_bounds__(4 * kBiasRows) void column_sum_final_kernel(BiasSum b)
{
    __shared__ float4 red[4 * kBiasRows];
    bias_sum_block<kBiasRows, BF16>(b, blockIdx.x, red);
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

hipError_t launch_column_sum(const BiasSum &b, int dtype, hipStream_t stream)
{
    if (b.Q < 0 || b.C4 < 1 || b.outside < 0 || b.extra < 1 || b.blocks < 1) return hipErrorInvalidValue;
    if (dtype == LBP_BF16) return LBP_LAUNCH_KERNEL(column_sum_final_kernel<true>, dim3(b.blocks), 4 * kBiasRows, 0, stream, b);
    return LBP_LAUNCH_KERNEL(column_sum_final_kernel<false>, dim3(b.blocks), 4 * kBiasRows, 0, stream, b);
}

}  // namespace lbp
