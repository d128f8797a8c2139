// Grouped launches that fit the device with one workgroup per compute unit: rings of 4 stages, read a whole stage
// ahead by 64-row input gradients (64 images 768 -> 3072 r = 4 21.8 -> 20.4 us; weight gradients beside them only take power).
#include "gemm_mfma_pair_impl.h"

namespace lbp {

hipError_t mfma_pair_w8_deep(const mfma::Params &x, int bm_x, GemmOut out_x, int lp_x, int splits_x, const mfma::Params &w,
                             int splits_w, hipStream_t s, bool w_leads, const BiasSum *bias)
{
    if (bm_x == 128) return mfma::pair_rings<128, mfma::ring(4, 64), mfma::ring(4, 64)>(x, out_x, lp_x, splits_x, w, splits_w, s, w_leads, bias);
    if (bm_x == 64) return mfma::pair_rings<64, mfma::ring(4, 64, true), mfma::ring(4, 64)>(x, out_x, lp_x, splits_x, w, splits_w, s, w_leads, bias);
    return hipErrorInvalidValue;
}

}  // namespace lbp
