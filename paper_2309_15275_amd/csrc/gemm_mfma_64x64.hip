// Instantiations of the bf16 matrix-core GEMM for 64 x 64 output tiles (2 x 2 wavefronts), for
// layers with few channels: a 128-wide tile would be mostly empty there.  Rings of 3 stages, three workgroups per
// compute unit, or of 2, four of them.
#include "gemm_mfma_impl.h"

namespace lbp {

hipError_t mfma_tile_64x64(const mfma::Params &p, bool a_kfast, GemmOut out, int lp, int splits, bool deep, hipStream_t s)
{
    if (deep) return mfma::launch_tile<64, 64, 2, 2, mfma::ring(3, 64), true>(p, a_kfast, out, lp, splits, s);
    return mfma::launch_tile<64, 64, 2, 2, mfma::ring(2, 64), true>(p, a_kfast, out, lp, splits, s);
}

}  // namespace lbp
