// Host side of the bf16 matrix-core GEMM: parameter set-up and the choice of tile shape.
#include <atomic>
#include <cmath>
#include <cstdlib>

#include "gemm_mfma_impl.h"

namespace lbp {
// Tile counters of the split reductions that combine inside a launch: zero whenever no such launch is
// running (the device image loads them as zeros and every launch leaves them so).  Each device has its
// own copy, found on first use.  Launches that overlap in time on one device must not both use them.
static __device__ unsigned join_counters[kJoinMaxTiles * kCounterPitch];

unsigned *join_counter_ptr()
{
    static std::atomic<unsigned *> ptrs[kMaxLaunchDevices] = {};       // (racing threads store the same value)
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxLaunchDevices) return nullptr;
    unsigned *found = ptrs[dev].load(std::memory_order_acquire);
    if (!found) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(join_counters)) != hipSuccess) return nullptr;
        found = static_cast<unsigned *>(ptr);
        ptrs[dev].store(found, std::memory_order_release);
    }
    return found;
}

int device_cus()
{
    static std::atomic<int> known{0};
    int cus = known.load(std::memory_order_relaxed);
    if (cus == 0) {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
            cus = v;
        else
            cus = 256;
        known.store(cus, std::memory_order_relaxed);
    }
    return cus;
}

namespace {

int round_up(int v, int m) { return (v + m - 1) / m * m; }

typedef hipError_t (*TileLaunch)(const mfma::Params &, bool, GemmOut, int, int, bool, hipStream_t);

// same order as kGemmTiles
const TileLaunch kLaunch[kNumGemmTiles] = {mfma_tile_128x128, mfma_tile_64x128, mfma_tile_128x256,
                                           mfma_tile_256x256, mfma_tile_128x128, mfma_tile_64x128, mfma_tile_64x64,
                                           mfma_tile_256x192, mfma_tile_256x128};

// Which ring a launch of `blocks` workgroups takes.  A longer one hides more of the way from memory, a shorter one lets
// more workgroups share a compute unit and overlap their epilogues and waits: the longer one pays while all
// workgroups are resident anyway (2048 x 768 x 3072 on 128 x 128, 96 of them: 31.5 -> 21.0 us; 4096 x 4096 x 1024, 1024 of
// them: 40 us against 51).
bool deep_ring(int tile, long blocks)
{
    if (tile == kTile128Deep) return true;
    if (tile == kTile64Shallow) return false;
    const int per_unit = tile == kTile128 ? 1 : tile == kTile64 ? 2 : 3;
    return blocks <= (long)per_unit * device_cus();
}

}  // namespace

bool gemm_can_fuse_unproject(const BasisPlan &plan, int dtype, GemmPath path)
{
    if (path == GemmPath::kSimple || dtype != LBP_BF16) return false;
    if (plan.patch != 4 && plan.patch != 8) return false;
    // Up to 16 pooled coefficients per channel the epilogue expands them with the register
    // butterfly; beyond that (selections that cannot be pooled) an 8 x 8 patch goes through the
    // matrix-core epilogue.  r <= patch^2 <= 64 always fits the smallest tile.
    return gemm_unproject_pooled(plan) || plan.patch == 8;
}

bool gemm_unproject_pooled(const BasisPlan &plan)
{
    return (plan.patch >> plan.mh) * (plan.patch >> plan.mw) <= 16;
}

namespace {

// Which tiles and slices each of the 8 XCDs works on: what is read by two XCDs comes twice from beyond their L2s, where all
// units together get about 7 TB/s (27 bytes a ns a unit; a 128 x 128 step wants 73).  Two ways, by the bytes an XCD reads:
//   * blocks: the XCDs in xcd_s groups that share out the slices of the reduction, the tiles of an XCD an xcd_a x xcd_b block;
//   * runs: an XCD takes an equal run of all workgroups, slice by slice, for counts that do not divide.  A weight gradient of
//     36 tiles in 7 slices is 0.9 of one slice per XCD then, where tile numbers dealt out round-robin had every XCD read nearly
//     both operands: 131072 tokens 768 x 768 at r = 16 71 -> 50 us (800 -> 120 MB read), 3072 x 768 over 16384 tokens
//     82 -> 72.
// Slices that join inside the launch are neighbours on one XCD, whose own L2 then holds their parts (8192 tokens 1024 -> 4096 r = 4, the
// input gradient alone in 4 slices: dealt out over the XCDs 21.0 us, on one 17.8); only where an XCD's run ends inside a tile,
// once per XCD, do that tile's slices lie on two.
void share_out(mfma::Params &p, int splits, int bn, bool joined)
{
    const long T = (long)p.tiles_m * p.tiles_n;
    p.count = (int)(T * splits);
    p.xcd_a = p.xcd_b = p.xcd_s = 0;
    double best = 1e300;
    for (int xs = 1; xs <= (joined ? 1 : 8); xs *= 2) {
        if (splits % xs || T * xs % 8) continue;
        for (int xb = 1; xb <= p.tiles_n; ++xb) {
            if (p.tiles_n % xb || (T * xs / 8) % xb) continue;
            const long xa = T * xs / 8 / xb;
            if (xa > p.tiles_m || p.tiles_m % xa) continue;
            const double bytes = ((double)xa * p.bm_step + (double)xb * bn) / xs;      // times K * 2 bytes
            if (bytes < best) {
                best = bytes;
                p.xcd_a = (int)xa;
                p.xcd_b = xb;
                p.xcd_s = xs;
            }
        }
    }
    const double run = p.count / 8.0 / (joined ? splits : 1), slices = fmax(1.0, run / T);
    double best_run = 1e300;
    p.run_band = 1;
    for (int h = 1; h <= p.tiles_m && h <= 64; ++h) {       // rows of tiles of a band; a run covers h x cols of them, or whole bands
        const double cols = fmin(run / h + 1.0, (double)p.tiles_n), rows = fmin((double)p.tiles_m, h * fmax(1.0, run / h / p.tiles_n));
        const double bytes = (rows * p.bm_step + cols * bn) * (joined ? 1.0 : slices / splits);
        if (bytes < best_run) {
            best_run = bytes;
            p.run_band = h;
        }
    }
    if (best_run < 0.8 * best) {       // (a tenth or two is within what the estimate of a run is worth)
        p.xcd_a = 0;
        p.xcd_s = joined ? splits : 1;
    }
}

// Checks one product, picks its tile and fills the kernel parameters.
hipError_t prepare(const GemmArgs &a, int *tile_out, mfma::Params *out, int *lp_out)
{
    if (a.dtype != LBP_BF16) return hipErrorInvalidValue;
    // rows of a k-fast A are clamped one by one (any M); a k-slow A and B are read in 8-element pieces
    if (a.M < (a.a_kfast ? 1 : 8) || a.N < 8 || a.K < 1) return hipErrorInvalidValue;
    if (a.N % 8 || a.ldb % 8 || a.lda % 8 || (a.a_kfast ? a.K % 8 : a.M % 8)) return hipErrorInvalidValue;
    // split reductions: fp32 slices for a reduction kernel, or a fused reverse projection whose slices combine in the launch
    if (a.out != GemmOut::kF32 && a.splits != 1 && !(a.out == GemmOut::kUnproject && a.join_parts && a.splits <= 16))
        return hipErrorInvalidValue;
    int tile = options().gemm_tile;     // testing: force one tile shape for every product
    if (tile >= 0 && a.out == GemmOut::kUnproject &&
        (!kGemmTiles[tile].fused || (tile == kTileWide && a.splits > 1) || (a.plan && !gemm_unproject_pooled(*a.plan) && kGemmTiles[tile].bn < 128)))
        tile = -1;
    if (tile < 0) tile = a.tile;
    if (tile < 0 || tile >= kNumGemmTiles) {
        const bool fused = a.out == GemmOut::kUnproject;
        tile = plan_gemm(a.M, a.N, a.K / a.splits, a.out == GemmOut::kF32 ? 4 : 2, false,
                         fused && a.plan ? a.plan->r : 0, fused && a.plan ? a.plan->patch : 0, device_cus(),
                         fused && a.plan && !gemm_unproject_pooled(*a.plan)).tile;
    }
    const GemmTileInfo &t = kGemmTiles[tile];

    mfma::Params p{};
    p.A = (const unsigned short *)a.A;
    p.B = (const unsigned short *)a.B;
    p.M = a.M; p.N = a.N; p.K = a.K;
    p.lda = (int)a.lda; p.ldb = (int)a.ldb;
    p.k_per_split = round_up((a.K + a.splits - 1) / a.splits, mfma::BK);
    p.bm_step = t.bm;
    p.tiles_n = (a.N + t.bn - 1) / t.bn;
    p.C = a.C;
    p.scale = a.scale;
    p.store_bf16 = a.out == GemmOut::kBF16 ? 1 : 0;
    int lp = 0;
    if (a.out == GemmOut::kUnproject) {
        if (!a.plan || !a.a_kfast || !t.fused || a.plan->r > t.bm || !gemm_can_fuse_unproject(*a.plan, a.dtype, GemmPath::kAuto))
            return hipErrorInvalidValue;
        const BasisPlan &bp = *a.plan;
        lp = bp.log2p;
        p.r = bp.r; p.mh = bp.mh; p.mw = bp.mw;
        p.bm_step = a.tile_step > 0 && tile == a.tile ? a.tile_step : fused_tile_step(t, a.M, a.N, a.K, bp.r, bp.patch, device_cus());
        if (p.bm_step > t.bm || p.bm_step % bp.r) return hipErrorInvalidValue;
        p.mfma_epilogue = gemm_unproject_pooled(bp) ? 0 : 1;
        if (p.mfma_epilogue && t.bn < 128) return hipErrorInvalidValue;
        for (int k = 0; k < 64; ++k) p.nat[k] = k < bp.r ? (unsigned char)bp.nat[k] : (unsigned char)0;
        if (!p.mfma_epilogue) {
            p.sel.mask = (unsigned)bp.pooled_mask;
            for (int j = 0; j < 16; ++j) p.sel.pos[j] = bp.pooled_pos[j];
        }
        if (a.extra_rows < 0 || a.extra_rows > a.M || (a.extra_rows > 0 && (a.extra < 1 || a.extra_rows % a.extra)) ||
            (a.M - a.extra_rows) % bp.r)
            return hipErrorInvalidValue;
        p.geom = make_geom(a.grid_h, a.grid_w, bp.patch, a.extra);
        p.Q = (a.M - a.extra_rows) / bp.r;     // = patches of the zero-padded grids
        p.extra_rows = a.extra_rows;
        p.extra = a.extra > 0 ? a.extra : 1;
    }
    p.tiles_m = (a.M + p.bm_step - 1) / p.bm_step;
    p.splits = 1;
    if (a.out == GemmOut::kUnproject && a.splits > 1) {
        if ((long)p.tiles_m * p.tiles_n > kJoinMaxTiles) return hipErrorInvalidValue;
        if ((long)(a.splits - 1) * p.k_per_split >= a.K) return hipErrorInvalidValue;       // no empty slice
        if ((size_t)p.tiles_m * p.tiles_n * a.splits * t.bm * t.bn * sizeof(float) > a.join_bytes) return hipErrorInvalidValue;
        p.splits = a.splits;
        p.parts = static_cast<float *>(a.join_parts);
        p.counters = join_counter_ptr();
        if (!p.counters) return hipErrorInvalidSymbol;
    }
    share_out(p, a.splits, t.bn, p.splits > 1);
    *tile_out = tile;
    *out = p;
    *lp_out = lp;
    return hipSuccess;
}

// Tiles of the grouped launch: 128x128 with 8 wavefronts for the weight gradient, that or 64x128
// with 8 wavefronts for the input gradient.
constexpr int kPairTileW = kTile128, kPairTileX0 = kTile128, kPairTileX1 = kTile64, kPairTileX2 = kTileWide;
// ... and 64x64 for both on thin layers
constexpr int kPairTileThin = kTileThin;

bool pair_tiles_ok(int tx, int tw)
{
    return (tw == kPairTileW && (tx == kPairTileX0 || tx == kPairTileX1 || tx == kPairTileX2)) || (tw == kPairTileThin && tx == kPairTileThin);
}

}  // namespace

bool gemm_join_supported(const GemmArgs &a, GemmPath path)
{
    if (path == GemmPath::kSimple || a.out != GemmOut::kUnproject || a.splits < 2 || !a.plan || (a.plan->patch != 8 && a.plan->patch != 4)) return false;
    int tile, lp;
    mfma::Params p;
    if (prepare(a, &tile, &p, &lp) != hipSuccess) return false;
    return tile == kPairTileX0 || tile == kPairTileX1;
}

hipError_t launch_gemm_mfma(const GemmArgs &a, hipStream_t stream)
{
    int tile, lp;
    mfma::Params p;
    hipError_t e = prepare(a, &tile, &p, &lp);
    if (e != hipSuccess) return e;
    // slices of a fused product join inside the launch on the 8-wavefront 128-wide tiles only
    if (a.out == GemmOut::kUnproject && a.splits != 1 && tile != kPairTileX0 && tile != kPairTileX1) return hipErrorInvalidValue;
    return kLaunch[tile](p, a.a_kfast, a.out, lp, a.splits, deep_ring(tile, (long)p.tiles_m * p.tiles_n * a.splits), stream);
}

bool gemm_pair_supported(const GemmArgs &x, const GemmArgs &w, GemmPath path)
{
    if (path == GemmPath::kSimple) return false;
    if (x.dtype != LBP_BF16 || w.dtype != LBP_BF16 || !x.a_kfast || w.a_kfast) return false;
    if (w.out == GemmOut::kUnproject) return false;
    if (x.out == GemmOut::kUnproject && (!x.plan || (x.plan->patch != 8 && x.plan->patch != 4))) return false;
    int tx, tw, lp;
    mfma::Params p;
    if (prepare(x, &tx, &p, &lp) != hipSuccess || prepare(w, &tw, &p, &lp) != hipSuccess) return false;
    if (tw == kPairTileThin && x.out == GemmOut::kUnproject && (!gemm_unproject_pooled(*x.plan) || x.splits != 1)) return false;
    if (tx == kPairTileX2 && (x.out != GemmOut::kUnproject || x.splits != 1)) return false;
    return pair_tiles_ok(tx, tw);
}

hipError_t launch_gemm_pair(const GemmArgs &x, const GemmArgs &w, hipStream_t stream, const BiasSum *bias)
{
    int tx, tw, lpx, lpw;
    mfma::Params px, pw;
    hipError_t e = prepare(x, &tx, &px, &lpx);
    if (e != hipSuccess) return e;
    e = prepare(w, &tw, &pw, &lpw);
    if (e != hipSuccess) return e;
    if (!pair_tiles_ok(tx, tw) || !x.a_kfast || w.a_kfast || w.out == GemmOut::kUnproject ||
        (x.out == GemmOut::kUnproject && lpx != 3 && lpx != 2))
        return hipErrorInvalidValue;
    // the dispatch order decides when a workgroup runs, never what it computes
    const long blocks = (long)px.tiles_m * px.tiles_n * x.splits + (long)pw.tiles_m * pw.tiles_n * w.splits;
    const bool w_leads = options().gemm_group == 2 || weight_gradient_first(tw == kPairTileThin, blocks, px.k_per_split / mfma::BK,
                                                                           pw.k_per_split / mfma::BK, device_cus());
    if (tw == kPairTileThin) return mfma_pair_64x64(px, x.out, lpx, x.splits, pw, w.splits, deep_ring(tw, blocks), stream, w_leads, bias);
    return mfma_pair_w8(px, kGemmTiles[tx].bm, kGemmTiles[tx].bn, x.out, lpx, x.splits, pw, w.splits, deep_ring(tw, blocks), stream, w_leads, bias);
}

}  // namespace lbp
