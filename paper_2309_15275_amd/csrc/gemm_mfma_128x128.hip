// Instantiations of the bf16 matrix-core GEMM for 128 x 128 output tiles (2 x 4 wavefronts): a ring of 4 stages, one
// workgroup per compute unit, or of 2, two of them.
#include "gemm_mfma_impl.h"

namespace lbp {

hipError_t mfma_tile_128x128(const mfma::Params &p, bool a_kfast, GemmOut out, int lp, int splits, bool deep, hipStream_t s)
{
    // A whole stage ahead for the transposing reads of a weight gradient, and with the pooled epilogue or slices that join (8 images 16 x 16
    // 1024 -> 4096 r = 4 27.3 -> 26.8 us).  Other input gradients are slower so: 4096 x 1024 x 1024 10.55 against 10.7 us, 2048 x 1024 x 4096 25.8
    // against 26.5, 32 images 768 -> 3072 r = 36 30.4 against 30.9.
    if (deep) return mfma::launch_tile<128, 128, 2, 4, mfma::ring(4, 64, true), true, mfma::ring(4, 64)>(p, a_kfast, out, lp, splits, s);
    return mfma::launch_tile<128, 128, 2, 4, mfma::ring(2, 64), true>(p, a_kfast, out, lp, splits, s);
}

}  // namespace lbp
