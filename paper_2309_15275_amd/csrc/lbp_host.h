// Host-side logic of the LBP-WHT library: argument validation, basis bookkeeping and the
// small tables the kernels receive by value.  Plain C++, no HIP calls, so that every function
// here can run (and be tested) on a machine without a GPU.
#pragma once
#include <cstddef>
#include <cstdint>

#include "../../include/lbp_wht.h"

namespace lbp {

constexpr int kMaxPatch = 16;
constexpr int kMaxBases = kMaxPatch * kMaxPatch;

// Sylvester (natural-order) row index of the Walsh function with `s` sign changes, for an
// order-2^log2p transform: the Gray code of s, bit-reversed.
int sequency_to_natural(int s, int log2p);

// -1 if p is not one of 2, 4, 8, 16, else log2(p).
int patch_log2(int patch);

// Patches of a batch of H x W token grids.  A grid that is not a multiple of the patch is treated
// as zero-padded at its bottom and right edges up to the next multiple (the paper's own maps are
// 7 x 7 = 49 tokens, Section 3.3).
inline long patch_count(int N, int H, int W, int patch)
{
    return (long)N * ((H + patch - 1) / patch) * ((W + patch - 1) / patch);
}
inline bool grid_is_ragged(int H, int W, int patch) { return H % patch != 0 || W % patch != 0; }

// How the register form of a projection launch (wht_kernels.hip) takes either tensor.
struct ProjectionReads {
    bool runs[2];        // neighbouring workgroups go to one XCD (xcd_run)
    bool cached[2];      // tokens are read without the non-temporal hint
};
// words: 32-bit words of a token, items: patches * words of either tensor (0: there is none).
//
// runs.  Rows that are not whole 128-byte lines gain (341 calls of this form, runs over none: 0.987 in the mean, 0.90 to 1.05).  Where the patches
// are less than half full (64, 8, 8 and 1 tokens on a 9 x 9 grid) and the device holds the launch at a time, it matters more which of them
// a unit gets: every 32nd place with runs (an XCD's 32 units take its workgroups in turn), every 256th without, and where that is close to a whole
// number of images, always the same one.  The order further from that is taken: 50 such calls 0.987 of the time without runs, 0.996 with runs
// always (0.95 to 1.05; 80 images 9 x 9, 48 -> 840 r = 4 22.3 -> 21.2 us with runs, 48 -> 1000 22.4 -> 23.2).  Whole lines meet no neighbour
// and gain less: 0.996 in the mean of 75 calls of two tensors (0.955 to 1.017), 0.99 of 16 x 16 and 32 x 32 grids.  One tensor alone
// whose patches hang over the grid's edge gains 0.2 % in the mean of 92 calls that the device holds at a time and loses up to 3 % (layer of
// 64 sequences of 1 + 14 x 14 tokens, 768 -> 3072 r = 8: its projection of g_y 18.3 -> 19.6, the training step 112.0 -> 113.1), and keeps its order.
//
// cached.  Narrow rows that are not whole lines: neighbouring tokens and wavefronts share lines, to be found in the L1 (calls: 64 images
// 56 x 56, 48 -> 192 r = 8 35.5 -> 32.2 us, 72 -> 192 40.8 -> 35.7; 60 images 40 x 40, 248 -> 1000 r = 4 73.6 -> 67.4; 64 images 56 x 56,
// 48 -> 96 fp32 62.1 -> 58.0).  Past 256 words a row the projection still gains, but tokens that stay in the Infinity Cache take the place of W
// and of the outputs, and calls lose up to 25 % (86 images 27 x 27, 1512 -> 104 r = 4 94 -> 118).  So do large tensors in front of an input
// gradient (gx_follows), which is as large as x, the second tensor.  Calls, read so / with the hint, by MB (10^6 bytes): both narrow, x below 24 0.97 (62 calls),
// 24 to 64 1.02 (47, to 1.10), above 1.17 (8, to 1.29); x alone below 24 0.96 (27), to 48 0.99 (21), to 64 1.01, above 1.07 (13, to 1.26);
// gy alone 0.97 to 1.00 until it passes 64 or x 80, then 1.00 and 1.02 (to 1.12).  Without an input gradient they gain at every size
// that was measured, to 100 (33 calls 0.93), and so does the projection alone (90 images 31 x 31, 488 and 328 channels, 84 and 57 MB, 57.8 -> 55.6).
// A launch of one tensor does not know what follows and keeps the hint (128 images 48 x 48, 488 -> 48 with x^ kept 73 -> 86 without).
// Whole lines are read once: 5 % slower without the hint.  Where one tensor of two is read so, the kernel has both forms in its code, and a launch of few
// workgroups waits for that: below one a unit, or 64 of that tensor (32 with 4 x 4 patches), 1.003 of the time with the hint in the mean of
// 120 calls (0.92 to 1.13; 62 images 23 x 23, 64 -> 48 r = 2 13.1 -> 15.1), above 0.97 of 260 (0.83 to 1.05).
ProjectionReads plan_projection_reads(int H, int W, int patch, long words0, long items0, long words1, long items1, bool gx_follows);

// The same order in the matrix-core form (wht_mfma_kernels.hip), one tensor of C channels in a launch of `blocks` workgroups.  Rows that are not whole
// lines: 320 calls 0.994 of the time in the mean (0.90 to 1.05), but 30 with patches at most 9/16 full that the device holds at a time
// 1.004 (0.975 to 1.044).  Whole lines are level, 4096 channels 2 % slower.
bool matrix_projection_runs(int H, int W, int patch, int C, long blocks);

// Everything the projection kernels need to know about the selected bases, passed to them by
// value in the kernel arguments (no device copy, no host/device synchronisation).
//
// A 2-D basis (u, v) in sequency order is natural-order coefficient nat(u)*p + nat(v) of the
// length-p^2 Hadamard transform of the row-major flattened patch.  If every selected nat(u) has
// its `mh` lowest bits clear and every nat(v) its `mw` lowest bits clear, the wanted coefficients
// equal those of the (p>>mh) x (p>>mw) transform of the patch sum-pooled over 2^mh x 2^mw token
// groups; `pooled_mask`/`pooled_pos` describe the selection in that smaller transform.
struct BasisPlan {
    int32_t patch;
    int32_t log2p;
    int32_t r;
    int32_t mh, mw;                 // pooling levels along H and W (0..log2p)
    uint8_t nat[kMaxBases];         // nat[k]: natural-order index of basis k in the p^2 transform
    uint64_t pooled_mask;           // bit j set: pooled natural coefficient j is selected (p <= 8)
    uint8_t pooled_pos[64];         // pooled natural coefficient j -> its position k (p <= 8)
};

// Checks patch / r / basis_idx and fills `plan`.  Returns LBP_OK or the matching error.
int make_basis_plan(int patch, const int32_t *basis_idx, int r, BasisPlan *plan);

int select_bases(int patch, int r, int order, int32_t *basis_idx);

// Low-heuristic-error selection (Section 3.2): the r bases of largest energy, by decreasing energy;
// equal energies keep the LP_L1 order.  energy has patch^2 entries indexed u*patch + v.
int select_lhe(const double *energy, int patch, int r, int32_t *basis_idx);

// Element size in bytes of a dtype code, 0 if unknown.
size_t dtype_size(int dtype);

// Shape / dtype / divisibility checks shared by the entry points.  patch == 0 skips the patch
// related checks (full-rank backward).
int validate_shape(const lbp_shape_t *shape, int patch);

// One tensor of a projection call.
int validate_grid(int N, int H, int W, int C, int dtype, int patch);

// LBP_ERR_ALIGN unless every listed pointer is 16-byte aligned (NULL entries are skipped).
int validate_alignment(const void *const *ptrs, int n);

// [a, a+na) and [b, b+nb) overlap?
bool ranges_overlap(const void *a, size_t na, const void *b, size_t nb);

// Tile shapes of the bf16 matrix-core GEMM (gemm_mfma_*.hip instantiates them in this order).  128x128 and 64x128 choose
// their ring of LDS stages by the size of the launch; the entries before them always take the named one and are there to be
// asked for (LBP_GEMM_TILE).
struct GemmTileInfo {
    int bm, bn;        // output tile of one workgroup
    bool fused;        // has the fused reverse-projection epilogue
    double slowdown;   // measured factor over the simple cost model below
    int max_n;         // only offered to products with at most this many columns (0: any)
    const char *name;  // for diagnostics
    bool whole_k = false;   // only offered to products the caller will not split along the reduction
    bool asked_only = false;   // the planner does not choose it
};
constexpr int kNumGemmTiles = 9, kAskableGemmTiles = 8;      // (the rest is for the planner alone)
constexpr int kTile128Deep = 0, kTile64Shallow = 1, kTileWide = 2, kTile128 = 4, kTile64 = 5, kTileThin = 6, kTileTall = 8;
extern const GemmTileInfo kGemmTiles[kNumGemmTiles];

// How one matrix product is run.
struct GemmPlan {
    int tile;          // index into kGemmTiles
    int splits;        // split-K slices (1 = the kernel writes the final output itself)
    double est_us;     // cost-model estimate, for diagnostics
};

// Picks tile shape and split-K factor for C[M][N] = A * B with reduction length K.
//   out_elem_bytes  size of one output element when the kernel stores the result itself
//   allow_split     the caller can reduce fp32 partial results afterwards
//   fused_r/patch   non-zero: the reverse projection is fused into the epilogue (rows are
//                   (patch, basis) pairs, r bases kept); implies no split
// The model: a compute unit takes in about 20 bytes a clock from L2 however many loads are in
// flight, so a workgroup's time is its operand and output bytes over that rate (or its matrix-core
// time if larger), and the workgroups run in ceil(count / compute units) rounds.
// fused_wide: the fused epilogue is the matrix-core one, which needs a 128-column tile.
// only_tile >= 0: consider that tile shape alone (est_us is 1e300 / clock when it cannot run the product); kAnyButWide: all but kTileWide.
constexpr int kAnyButWide = -2;
GemmPlan plan_gemm(long M, long N, long K, int out_elem_bytes, bool allow_split, int fused_r,
                   int fused_patch, int num_cus, bool fused_wide = false, int only_tile = -1, bool filled = false);

// Rows a tile with the fused reverse projection advances by: whole patches of r rows, as many as fit up to 16; beyond
// that (small r) as many as make the launch shortest, because one workgroup stores its tokens at about 45 GB/s: at r = 2
// the 32 patches of a 64 x 128 tile are 0.5 MB, 12 us, while most of the device is idle.
// filled: something else fills the device beside this product, so all patches that fit.
int fused_tile_step(const GemmTileInfo &ti, long M, long N, long K, int r, int patch, int num_cus, bool filled = false);

// Workgroups the plan launches for an M x N output (fused_r, fused_patch as in plan_gemm).
long gemm_workgroups(const GemmPlan &g, long M, long N, long K, int fused_r, int fused_patch, int num_cus, bool filled = false);

// Workspace layout of one backward call; offsets in bytes from the workspace base, each
// 256-byte aligned.  Sizes of 0 mean "not used".
struct WorkspacePlan {
    size_t gy_r, x_r, gx_r, splitk;   // offsets
    size_t total;                      // bytes
    GemmPlan gw;                       // the weight-gradient product
    GemmPlan gx;                       // the input-gradient product
    bool gx_fused;                     // reverse projection fused into that product's epilogue
    int gx_step;                       // ... and the rows of whole patches a tile advances by
    int f32_rows_x, f32_rows_w;        // fp32: rows of the tiles of either product
    bool grouped;                      // both products run in one launch (tiles chosen for that)
    bool or_apart;                     // ... in slices; two launches come next where there is no room for those
    bool gx_coef16;                    // not fused: the product stores its coefficients as bf16 in one
                                       // piece (no split-K) and the reverse projection reads those
    int gx_join;                       // fused and grouped: slices of the input-gradient product's reduction that
                                       // combine inside the launch (1: none); their partial tiles live at gx_r,
    size_t gx_join_bytes;              // in this many bytes
    size_t gx_parts;                   // fp32: offset of the input-gradient product's parts (bf16: they live at gx_r)
    size_t gw_join_bytes;              // fp32: slices of the weight-gradient product join too (gw.splits of them), at splitk
};

// Tiles of a launch whose products are cut into slices that join inside it (one counter each).
constexpr int kMaxJoinedTiles = 16384;

// fp32 products in bf16 parts (gemm_f32_mfma.hip): tiles of 64 or 128 rows x 64, reduction steps of 32.
// Rows a tile of `rows` advances by: whole patches of r rows (r = 0: all of them), as many as fit unless a few would leave the
// stores of all tokens to a few workgroups (one workgroup stores a patch of 64 tokens x 64 channels in about 0.3 us, a step of 64
// rows takes 0.45): at r = 1 a full tile is 64 patches, 1 MB of tokens.
int f32_tile_step(long M, long N, long K, int r, int patch, int num_cus, int rows = 64);
long f32_tiles(long M, long N, int step);
struct F32Cut {
    int splits_x, splits_w;
    double us;           // estimated length of the launch
};
// Slices of the two products of one launch (0 tiles: absent) and an estimate of how long it takes: of the ways to cut both into slices of
// about one length, none shorter than 6 steps, at most max_splits a tile, the one whose longest unit ends first by a model of steps,
// joins and epilogues.  end_x: what a tile's epilogue takes.
constexpr int kMaxF32Splits = 16;
F32Cut plan_f32_products(long tiles_x, long K_x, long tiles_w, long K_w, int num_cus, int max_splits = kMaxF32Splits, int rows_x = 64,
                         int rows_w = 64, double end_x = 0.0);
// Workspace of an fp32 call on those kernels; patch 0: the exact backward.  fuse: p^-1 in the product's epilogue.
int plan_workspace_f32(const lbp_shape_t *shape, int patch, int r, bool fuse, bool want_gx, bool want_gw, int extra,
                       WorkspacePlan *ws, int num_cus, int max_splits = kMaxF32Splits);

// Arrival counters of the one-pass energy kernels belong to a workspace, as the partial sums that they guard do: calls that overlap
// in time on different workspaces must not count each other's workgroups.  Set 0 is the library's own workspace, the others are
// given out to callers' workspaces by address, for good (a recorded graph may come back to one at any time); -1: all are taken.
struct CounterSets {
    static constexpr int kSets = 16;
    const void *owner[kSets] = {};
    int of(const void *workspace);      // (guarded by the caller's lock)
};

// Rows of partial sums of the bias gradient where the projection does not leave them: 8 tokens or more each, at most 1024 (one
// workgroup per row and 1024 channels; the rows are read once more).
inline long bias_sum_rows(long tokens) { return tokens < 8 * 1024 ? (tokens + 7) / 8 : 1024; }

// Where such rows (of patches or of tokens, `bytes` of them) lie while workgroups beside both products add them up: on the x^ of the plan if
// they fit there (a call with a bias gradient brings its x^ along), else behind the products' memory.
inline size_t bias_sums_beside(const WorkspacePlan &ws, size_t bytes)
{
    return bytes <= ws.gx_r - ws.x_r ? ws.x_r : (ws.total + 255) / 256 * 256;
}

// num_cus: compute units of the device (the GEMM plans depend on it); pass 256 when unknown.
// can_fuse: the selection allows the fused reverse projection (false gives the larger workspace);
// force_fuse: take it whenever allowed instead of comparing estimates; fused_wide: see plan_gemm;
// allow_group: the caller wants both gradients and can launch the two products as one grid;
// extra: tokens per image in front of the grid (tensors are [N][extra + H*W][C]);
// coef16: 1 = the caller has a reverse projection that reads bf16 coefficients (gx_coef16 may be
// chosen), 2 = take it whenever the reverse projection is not fused, 0 = never.
// gx_join: 0 = choose the number of joined slices of a fused, grouped input-gradient product, n = take n.
// smallest: nothing cut into slices, the reverse projection fused if it can be: no plan of the same call needs less memory.
int plan_workspace(const lbp_shape_t *shape, int patch, int r, int num_cus, bool can_fuse,
                   bool force_fuse, WorkspacePlan *ws, bool fused_wide = false, bool allow_group = false,
                   int extra = 0, int coef16 = 0, int gx_join = 0, bool smallest = false);

// Estimated length in microseconds of a grouped launch on `num_cus` compute units: n_x workgroups of the
// input-gradient product (cost_x each) and n_w of the weight-gradient product (cost_w each), dispatched
// in that order (or the other way round), the i-th workgroup to unit i mod num_cus, workgroups on one
// unit sharing it.
double grouped_launch_estimate(long n_x, double cost_x, long n_w, double cost_w, int num_cus, bool w_first);

// Whether a grouped launch of `blocks` workgroups dispatches the weight gradient's first; the planner and the launch ask this same
// question.  steps_x, steps_w: steps of 64 of a workgroup of either product.
// When the launch has more workgroups than the device holds at once (two of these per compute unit), those with the higher indices start
// late, and the launch ends with them: the product whose workgroups take longer goes first.  The rule counts their steps.  That is the weight
// gradient unless the input gradient's workgroups have clearly more of them, because its tiles end with long bursts of stores, behind which
// the loads of the weight gradient's queue.  Products of 109 random layers, weight gradient first over last: 77 where the rule puts it first
// 0.972 of the time in the mean (0.80 to 1.09; 8 lose more than 3 %, most of them with about equal steps), 32 where it goes last 1.21
// (0.98 to 1.37).  20 of those 32 have input gradients on 64-row tiles, whose steps are a third shorter than the others': such launches are only
// planned with slices that join, 3 and more times as long as the weight gradient's.  131072 tokens 768 -> 768 at r = 4, 8 and 16 (12 steps against 19, 37,
// 74) 67 us against 79, 84 / 96, 125 / 146; 16384 tokens 768 -> 3072 with the 16 bases of smallest sequency sum (48 against 22) 78 / 67, with
// 20 bases 87 / 77; 6996 tokens 2560 -> 2640 r = 8 (42 against 16) 68 / 57; 13650 tokens 2608 -> 2672 r = 10 (42 against 39) 126 / 130.
// Where everything is resident the order makes 4 % either way: those launches, and thin layers, keep the input gradient first.
inline bool weight_gradient_first(bool thin, long blocks, long steps_x, long steps_w, int num_cus)
{
    return !thin && blocks > 2L * num_cus && 4 * steps_x < 5 * steps_w;
}

const char *status_string(int code);

// Kernel-choice switches (tests and measurement; see lbp_set_option in the public header).
struct Options {
    int wht_path = 0;          // 0 chosen per selection, 1 generic, 2 register, 3 matrix-core
    int gemm_simple = 0;       // 1: plain cross-check products
    int gemm_tile = -1;        // >= 0: one tile shape for every product
    int fuse_unproject = -1;   // -1 planner, 0 never, 1 wherever the kernel supports the selection
    int gemm_group = 1;        // 0: the two products of a call in separate launches; 2: one launch, weight gradient first
    int gx_coef = 1;           // 1 planner, 0 fp32 slices, 2 bf16 wherever the kernels allow
    int gx_join = 0;           // 0 planner, 1..8: that many joined slices wherever the grouped fused launch runs
};
// The current switches; the first call reads the LBP_* environment variables, once per process.
Options options();
// One switch by name; value NULL restores the default.  LBP_OK, LBP_ERR_NULL or LBP_ERR_OPTION.
int set_option(const char *name, const char *value);

}  // namespace lbp
