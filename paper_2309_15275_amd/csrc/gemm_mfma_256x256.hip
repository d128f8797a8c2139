// Instantiations of the bf16 matrix-core GEMM for 256 x 256 output tiles (2 x 4 wavefronts), a ring of 5 stages of 32 (all of a unit's LDS).
#include "gemm_mfma_impl.h"

namespace lbp {

hipError_t mfma_tile_256x256(const mfma::Params &p, bool a_kfast, GemmOut out, int lp, int splits, bool, hipStream_t s)
{
    return mfma::launch_tile<256, 256, 2, 4, mfma::ring(5, 32), false>(p, a_kfast, out, lp, splits, s);
}

}  // namespace lbp
