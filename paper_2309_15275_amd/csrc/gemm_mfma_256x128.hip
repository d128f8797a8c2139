// Instantiations of the bf16 matrix-core GEMM for 256 x 128 output tiles (4 x 2 wavefronts), a ring of 3 stages of 64, one workgroup per compute
// unit: for unfused products whose columns leave 128 x 256 tiles half empty (41616 rows 1136 -> 88 channels 32.7 us on 128 x 128 tiles, 29.1 so), and
// for the second of two products that finds its operand in the caches (plan_workspace).
#include "gemm_mfma_impl.h"

namespace lbp {

hipError_t mfma_tile_256x128(const mfma::Params &p, bool a_kfast, GemmOut out, int lp, int splits, bool, hipStream_t s)
{
    return mfma::launch_tile<256, 128, 4, 2, mfma::ring(3, 64), false>(p, a_kfast, out, lp, splits, s);
}

}  // namespace lbp
