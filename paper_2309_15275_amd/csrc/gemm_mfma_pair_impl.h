// The grouped launch (input-gradient product + weight-gradient product in one grid) on the 8-wavefront tiles, for one
// choice of rings (mfma::ring): STX and STW.
#pragma once
#include "gemm_mfma_impl.h"

namespace lbp {
namespace mfma {

template <int BMX, int BNX, int STX, int STW, int EPIX, int LPX, bool JOINX = false>
hipError_t pair_one(const Params &x, int splits_x, const Params &w, int splits_w, hipStream_t s, bool w_leads, const BiasSum *bias)
{
    return launch_pair<2, 4, STX, BMX, BNX, true, EPIX, LPX, STW, 128, 128, false, EPI_PLAIN, 0, JOINX>(x, splits_x, w, splits_w, s,
                                                                                                       w_leads, bias);
}

template <int BMX, int STX, int STW, int BNX = 128>
hipError_t pair_rings(const Params &x, GemmOut out_x, int lp_x, int splits_x, const Params &w, int splits_w, hipStream_t s,
                      bool w_leads, const BiasSum *bias)
{
    if (out_x == GemmOut::kUnproject) {
        if constexpr (BNX == 128) {
            if (splits_x != 1) {        // the slices of a tile combine inside the launch, the last one runs the epilogue
                if (!x.parts || !x.counters || x.splits != splits_x) return hipErrorInvalidValue;
                if (lp_x == 2) return pair_one<BMX, BNX, STX, STW, EPI_UNPROJECT, 2, true>(x, splits_x, w, splits_w, s, w_leads, bias);
                if (x.mfma_epilogue) return pair_one<BMX, BNX, STX, STW, EPI_UNPROJECT_MFMA, 3, true>(x, splits_x, w, splits_w, s, w_leads, bias);
                return pair_one<BMX, BNX, STX, STW, EPI_UNPROJECT, 3, true>(x, splits_x, w, splits_w, s, w_leads, bias);
            }
        }
        if (lp_x == 2) return pair_one<BMX, BNX, STX, STW, EPI_UNPROJECT, 2>(x, 1, w, splits_w, s, w_leads, bias);
        if (x.mfma_epilogue) return pair_one<BMX, BNX, STX, STW, EPI_UNPROJECT_MFMA, 3>(x, 1, w, splits_w, s, w_leads, bias);
        return pair_one<BMX, BNX, STX, STW, EPI_UNPROJECT, 3>(x, 1, w, splits_w, s, w_leads, bias);
    }
    if constexpr (BNX == 128) return pair_one<BMX, BNX, STX, STW, EPI_PLAIN, 0>(x, splits_x, w, splits_w, s, w_leads, bias);
    else return hipErrorInvalidValue;
}

}  // namespace mfma
}  // namespace lbp
