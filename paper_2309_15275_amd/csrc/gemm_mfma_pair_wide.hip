// Grouped launches with input gradients on 128 x 256 tiles, two workgroups of either product per compute unit: both gradients of 5376
// rows (13 x 8 patches, r = 22) 584 -> 904 channels 69.8 us on 128 x 128 tiles, 59.4 so.
#include "gemm_mfma_pair_impl.h"

namespace lbp {

hipError_t mfma_pair_w8_wide(const mfma::Params &x, GemmOut out_x, int lp_x, int splits_x, const mfma::Params &w, int splits_w,
                             hipStream_t s, bool w_leads, const BiasSum *bias)
{
    if (splits_x != 1) return hipErrorInvalidValue;
    return mfma::pair_rings<128, mfma::ring(3, 32), mfma::ring(2, 64), 256>(x, out_x, lp_x, 1, w, splits_w, s, w_leads, bias);
}

}  // namespace lbp
