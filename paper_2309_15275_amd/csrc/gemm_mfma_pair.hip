// Instantiations of the grouped launch (input-gradient product + weight-gradient product in one
// grid) for the tiles the planner gives the low-rank products: the 8-wavefront ones, two workgroups per compute unit (124
// registers at most), and 64 x 64 for layers with few channels.
#include "gemm_mfma_pair_impl.h"

namespace lbp {
namespace {
using namespace mfma;

template <int ST, int EPIX, int LPX>
hipError_t thin(const Params &x, int splits_x, const Params &w, int splits_w, hipStream_t s, bool w_leads, const BiasSum *bias)
{
    return launch_pair<2, 2, ST, 64, 64, true, EPIX, LPX, ST, 64, 64, false, EPI_PLAIN, 0>(x, splits_x, w, splits_w, s, w_leads, bias);
}

template <int ST>
hipError_t thin_ring(const Params &x, GemmOut out_x, int lp_x, int splits_x, const Params &w, int splits_w, hipStream_t s,
                     bool w_leads, const BiasSum *bias)
{
    if (out_x == GemmOut::kUnproject) {
        if (splits_x != 1 || x.mfma_epilogue) return hipErrorInvalidValue;
        if (lp_x == 2) return thin<ST, EPI_UNPROJECT, 2>(x, 1, w, splits_w, s, w_leads, bias);
        return thin<ST, EPI_UNPROJECT, 3>(x, 1, w, splits_w, s, w_leads, bias);
    }
    return thin<ST, EPI_PLAIN, 0>(x, splits_x, w, splits_w, s, w_leads, bias);
}
}  // namespace

hipError_t mfma_pair_64x64(const mfma::Params &x, GemmOut out_x, int lp_x, int splits_x, const mfma::Params &w, int splits_w,
                           bool deep, hipStream_t s, bool w_leads, const BiasSum *bias)
{
    if (deep) return thin_ring<ring(3, 64)>(x, out_x, lp_x, splits_x, w, splits_w, s, w_leads, bias);
    return thin_ring<ring(2, 64)>(x, out_x, lp_x, splits_x, w, splits_w, s, w_leads, bias);
}

hipError_t mfma_pair_w8_deep(const mfma::Params &x, int bm_x, GemmOut out_x, int lp_x, int splits_x, const mfma::Params &w,
                             int splits_w, hipStream_t s, bool w_leads, const BiasSum *bias);
hipError_t mfma_pair_w8_wide(const mfma::Params &x, GemmOut out_x, int lp_x, int splits_x, const mfma::Params &w, int splits_w,
                             hipStream_t s, bool w_leads, const BiasSum *bias);

hipError_t mfma_pair_w8(const mfma::Params &x, int bm_x, int bn_x, GemmOut out_x, int lp_x, int splits_x, const mfma::Params &w,
                        int splits_w, bool deep, hipStream_t s, bool w_leads, const BiasSum *bias)
{
    if (bn_x == 256) return mfma_pair_w8_wide(x, out_x, lp_x, splits_x, w, splits_w, s, w_leads, bias);
    if (deep) return mfma_pair_w8_deep(x, bm_x, out_x, lp_x, splits_x, w, splits_w, s, w_leads, bias);
    if (bm_x == 128) return mfma::pair_rings<128, mfma::ring(2, 64), mfma::ring(2, 64)>(x, out_x, lp_x, splits_x, w, splits_w, s, w_leads, bias);
    if (bm_x == 64) return mfma::pair_rings<64, mfma::ring(3, 64), mfma::ring(2, 64)>(x, out_x, lp_x, splits_x, w, splits_w, s, w_leads, bias);
    return hipErrorInvalidValue;
}
}  // namespace lbp
