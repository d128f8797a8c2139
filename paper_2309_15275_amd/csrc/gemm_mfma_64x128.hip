// Instantiations of the bf16 matrix-core GEMM for 64 x 128 output tiles (2 x 4 wavefronts): a ring of 3 stages, two
// workgroups per compute unit, or of 2, three of them.
#include "gemm_mfma_impl.h"

namespace lbp {

hipError_t mfma_tile_64x128(const mfma::Params &p, bool a_kfast, GemmOut out, int lp, int splits, bool deep, hipStream_t s)
{
    if (deep) return mfma::launch_tile<64, 128, 2, 4, mfma::ring(3, 64), true>(p, a_kfast, out, lp, splits, s);
    return mfma::launch_tile<64, 128, 2, 4, mfma::ring(2, 64), true>(p, a_kfast, out, lp, splits, s);
}

}  // namespace lbp
