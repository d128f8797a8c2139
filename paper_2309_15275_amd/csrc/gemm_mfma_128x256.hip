// Instantiations of the bf16 matrix-core GEMM for 128 x 256 output tiles (2 x 4 wavefronts), a ring of 3 stages of 32, two workgroups per
// compute unit.  Against 128 x 128 tiles, two workgroups a unit as well, an output element costs three quarters of the operand bytes and two
// thirds of the LDS reads (64 x 64 a wavefront), and loads have twice the time to arrive; products of plain bf16 output, 128 x 128 / 128 x 256:
// 4096 x 4096 x 1024 36.5 / 33.6 us, 32768 x 768 x 768 50.5 / 43.8, 4608 x 3072 x 768 27.1 / 25.1, 16384 x 768 x 3072 90 / 80.  256 x 128 tiles, whose
// reduction-fast operand comes in half lines in steps of 32, gain nothing (36.8, 49.9, 27.1, 94).  128 registers: what the epilogue
// spills is not in the loop.
#include "gemm_mfma_impl.h"

namespace lbp {

hipError_t mfma_tile_128x256(const mfma::Params &p, bool a_kfast, GemmOut out, int lp, int splits, bool, hipStream_t s)
{
    return mfma::launch_tile<128, 256, 2, 4, mfma::ring(3, 32), true>(p, a_kfast, out, lp, splits, s);
}

}  // namespace lbp
