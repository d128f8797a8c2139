// Instantiations of the bf16 matrix-core GEMM for 256 x 192 output tiles (4 x 2 wavefronts), a ring of 5 stages of 32 (a stage is one
// sub-step, read ahead as a whole: in halves of A's rows the exact input gradient of 16384 tokens 768 -> 3072 takes 74 us, not 68).
#include "gemm_mfma_impl.h"

namespace lbp {

hipError_t mfma_tile_256x192(const mfma::Params &p, bool a_kfast, GemmOut out, int lp, int splits, bool, hipStream_t s)
{
    return mfma::launch_tile<256, 192, 4, 2, mfma::ring(5, 32, true), false>(p, a_kfast, out, lp, splits, s);
}

}  // namespace lbp
