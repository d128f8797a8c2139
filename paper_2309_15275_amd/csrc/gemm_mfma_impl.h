// bf16 matrix-core GEMM kernel template for gfx950 (fp32 accumulation); instantiated per tile
// shape by the gemm_mfma_*.hip files.
//
// One workgroup owns a BM x BN tile of the output and walks the reduction in steps of 64 or 32.
//   * Global memory -> LDS directly (16 bytes a lane), into a ring of STAGES stages; step s+STAGES is requested as soon as
//     nobody reads step s any more.  One barrier per step: by then all fragments of the step are in registers.  Fragments
//     are read while earlier ones are multiplied, across steps too: a sub-step of 32 (or half of one) ahead, placing the barrier
//     before the step's last part, or a whole stage ahead, the barrier in front of the step and its loads spread between the matrix
//     instructions.  Rows and columns past the edge of a matrix are clamped
//     to the last valid ones (they only feed outputs that are never stored); only a final partial step of the
//     reduction zero-fills, through registers.  Against staging through registers (two LDS stages, two steps of loads in
//     registers, a barrier at every step's end) with the same tiles and bit-identical results, one product alone:
//     8192^3 on 256 x 256 972 -> 814 us (1.35 PFLOP/s); 16384 x 768 x 3072 on 256 x 192 72 -> 63 us; 3072 x 768 x 2048 on
//     128 x 128 22.3 -> 16.9 us; 2048 x 768 x 3072 on 64 x 128 20.5 -> 16.8 us.
//   * What bounds a step: everything about equally.  In clocks of a 128 x 128 x 64 step (8 wavefronts): matrix instructions 512,
//     taking in 32 KB 512 (64 bytes a clock; 55-60 are reached), LDS reads 413 and as much again as 200 for the arriving
//     data; each of them alone in this loop takes 544, 712 and 600, all together 790-820 with one workgroup a unit and 670
//     with two, while the units' clock falls from 2.3 to 1.6-1.9 GHz.  So the loop gains little from hiding any one
//     of them better.  What did gain: a whole stage of lookahead for a lone weight gradient on 128 x 128 tiles (both operands through
//     transposing reads, half as wide: 1024 x 4096 x 4096 32.9 -> 29.7 us in the loop, 990 -> 840 clocks a step), and five stages
//     of 32 instead of two of 64 for the 256-wide tiles, whose loads then have two steps to arrive, not one (both exact
//     products of 16384 tokens 768 -> 3072 157.0 -> 153 us).  The lookahead is also taken by 64-row input gradients of resident launches of both
//     products, whole or in slices (the launch 0 to 6.5 % shorter: 64 images 768 -> 3072 r = 4 21.8 -> 20.4 us), by the pooled epilogue and
//     slices that join on deep 128 x 128 tiles (level to 1.5 %), and by 256 x 192 tiles, where a stage of 32 is one sub-step (taken in halves of
//     A's rows instead, exact products are 3 to 11 % slower).  What did not gain: the lookahead for other input gradients on deep 128 x 128 tiles
//     (1 to 2.5 % slower), for the weight gradient in launches of both
//     products (faster, it only takes power from the input gradient, which ends last: 12608 tokens 768 -> 3072,
//     a layer's step 121.9 -> 123.6 us); 32-deep steps on 128 x 128 tiles (twice the barriers: 24 against 20 us for 48 steps); LDS
//     reads left in flight across the barrier (level); two groups of wavefronts half a step apart, one reading while the other multiplies
//     (28.7 -> 34.2 us for both products of 16384 tokens 768 -> 3072 r = 8).  A step of 64 takes (us, one workgroup a unit / two):
//     64 x 128 0.28-0.32 / 0.54-0.58; 128 x 128 0.41-0.50 / 0.77-0.92.
//   * Operands whose reduction index is contiguous in memory are stored [row][k] in LDS and read
//     back with 16-byte reads.  Operands whose reduction index is the slow axis (W, and both
//     operands of gW) are stored as they arrive, [k][row], and transposed on the way to the
//     matrix cores with ds_read_b64_tr_b16: within each group of 16 lanes, lane i supplies the
//     address of 4 consecutive elements of row k = i/4 starting at column 4*(i%4), and lane j
//     receives the 4 k-values of column j.  Two such reads give the 8 consecutive k-values per
//     lane that v_mfma_f32_16x16x32_bf16 takes.  Pieces of a row are permuted so that both access patterns spread over
//     all LDS banks.
//   * Each wavefront owns a (BM/WGM) x (BN/WGN) block of 32x32 accumulators, four 16 x 16 products each.  Long products are
//     bound by power: the units run at 1.7-1.8 of 2.4 GHz.  On random operands and nothing else the 16 x 16 x 32 form
//     holds 2.1-2.2 PFLOP/s, 32 x 32 x 16 1.9 (2.4 both on zeros).  With it the exact input gradient of 16384 tokens
//     3072 -> 768 takes 75.7 instead of 78.4 us, the weight gradient 81.4 instead of 83.5, both products of the 49-token
//     maps at r = 36 63.3 instead of 65.8, of 8192 tokens 1024 -> 4096 r = 16 40.8 instead of 42.2; short ones are level.
//     The operands are exchanged in the instruction, which makes the result's transpose: a lane then holds neighbouring
//     columns and writes 16 bytes at a time, to LDS and to memory.
//   * Epilogues: scaled fp32 store (per split-K slice), scaled bf16 store, or the reverse
//     projection of Eq. 7 fused in: the tile's rows are (patch, basis) pairs, the accumulators go
//     through LDS, and every lane expands the r coefficients of one (patch, channel pair) into
//     the p x p tokens of that patch with the same pooled butterfly the stand-alone kernel uses.
//   * Workgroups are numbered so that each of the 8 XCDs (private L2 each) works on a 2-D block of
//     tiles, or a run of slices and tiles, whose strips of A and B are the fewest bytes.
//   * A fused product with few tiles under a long reduction can cut the reduction into slices, one
//     workgroup each, that combine inside the launch (JOIN instantiations): see store_part below.
#pragma once
#include <type_traits>

#include "bias_device.h"
#include "device_utils.h"
#include "kernels.h"
#include "launch.h"
#include "wht_device.h"

namespace lbp {
namespace mfma {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef short i16x4_t __attribute__((ext_vector_type(4)));
typedef short i16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));     // (the reverse projection on the matrix cores)
typedef float f32x4_t __attribute__((ext_vector_type(4)));
// A 32 x 32 block of accumulators: four 16 x 16 products, [2 * row half + column half].  Transposed, so that a lane holds four
// neighbouring columns: element e is row lane % 16, column 4 * (lane / 16) + e of its half.
typedef f32x4_t acc_t[4];

#define LBP_LDS_PTR(T, p) ((__attribute__((address_space(3))) T *)(p))

constexpr int BK = 64;

// EPI_PLAIN: fp32 or bf16 store chosen at run time by Params::store_bf16 (grouped launches)
enum { EPI_F32 = 0, EPI_BF16 = 1, EPI_UNPROJECT = 2, EPI_UNPROJECT_MFMA = 3, EPI_PLAIN = 4 };

// One product (kernel arguments are kept small: see launch.h).
struct Plain {
    const unsigned short *A;
    const unsigned short *B;
    void *C;
    int M, N, K;
    int lda, ldb;
    int k_per_split;      // multiple of BK
    int bm_step;          // rows of the output one tile advances by (BM, or a multiple of r below BM)
    int tiles_m, tiles_n;
    int xcd_a, xcd_b;     // tiles of one XCD form an xcd_a x xcd_b block of the output,
    int xcd_s;            // and xcd_s groups of XCDs share out the slices of the reduction; or (xcd_a = 0)
    int run_band;         // an XCD's workgroups are a run of all, xcd_s slices at a time, tiles in bands of so many rows
    int count;            // tiles x slices
    float scale;
    int store_bf16;       // EPI_PLAIN: 1 stores bf16, 0 stores fp32 (slice by slice)
};

// ... with the reverse projection fused in
struct Params : Plain {
    GridGeom geom;
    struct {
        unsigned mask;           // pooled coefficients that are selected, and their rows (at most 16 in the pooled epilogue)
        unsigned char pos[16];
    } sel;
    int r, mh, mw;
    int extra_rows;       // rows of A after the Q*r (patch, basis) rows: tokens outside the grid, extra per image
    int extra;            // such tokens per image; their rows of the product are stored scaled by 1/patch^2
    int mfma_epilogue;    // 1: the selection cannot be pooled, Eq. 7 runs on the matrix cores in the epilogue
    long Q;               // number of patches
    unsigned char nat[64];   // natural (Sylvester) index of every selected basis (matrix-core epilogue, patch 8)
    // reduction split over `splits` workgroups per tile that combine inside the launch (JOIN kernels only)
    int splits;           // slices per tile
    float *parts;         // [tile][slice][BM * BN] partial accumulators
    unsigned *counters;   // one per tile (kCounterPitch apart), zero between launches
};

// (a class, not a condition in the kernels' signatures: those have to mangle alike on host and device)
template <int EPI> struct ParamsFor { typedef Plain type; };
template <> struct ParamsFor<EPI_UNPROJECT> { typedef Params type; };
template <> struct ParamsFor<EPI_UNPROJECT_MFMA> { typedef Params type; };
template <int EPI> using ParamsOf = typename ParamsFor<EPI>::type;

// Scheduling hint for one sub-step of the main loop: N matrix instructions with R LDS reads spread
// evenly over the first two thirds of them, so that the last have arrived when the next sub-step starts (ViT-B fc1 products
// 30.3 us spread over all, 29.1 so; the arguments of the builtin must be constants, hence the recursion).
template <int I, int N, int R>
__device__ __forceinline__ void interleave_mfma_with_lds_reads()
{
    if constexpr (I < N) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);          // one matrix instruction
        constexpr int upto = R * (I + 1) * 3 / (N * 2), before = R * I * 3 / (N * 2);
        constexpr int share = (upto < R ? upto : R) - (before < R ? before : R);
        if constexpr (share > 0) __builtin_amdgcn_sched_group_barrier(0x100, share, 0);      // its share of the LDS reads
        interleave_mfma_with_lds_reads<I + 1, N, R>();
    }
}

typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));     // 16 bytes, usable with the non-temporal builtins

// Where the patches of one tile lie: element index of their first token, tokens of the patch inside the grid.
struct PatchAt {
    size_t at;
    int hv, wv;          // 0: no such patch
};

__device__ __forceinline__ void locate_patches(const Params &p, int m0, int patches, PatchAt *at, int tid)
{
    for (int pt = tid; pt < patches; pt += blockDim.x) {
        const long q = (long)(m0 / p.r) + pt;
        PatchAt a{0, 0, 0};
        if (q < p.Q) {
            long img;
            int a0, b0;
            p.geom.origin(q, img, a0, b0);
            a.at = p.geom.token(img, a0, b0) * p.N;
            a.hv = p.geom.Ht - a0;
            a.wv = p.geom.Wt - b0;
        }
        at[pt] = a;
    }
}

// `count` patches of pooled tokens staged in LDS as bf16 rows [patch][nc][BN] -> tokens in memory, 16 bytes a lane.  A lane
// has the same piece of the same tokens in every patch, so that a store costs an LDS read and an addition.
template <int LP, int BN, int NT>
__device__ __forceinline__ void store_pooled(const unsigned char *stg, int count, int nc, const PatchAt *at, const Params &p, int n0,
                                             int tid)
{
    constexpr int P = 1 << LP, P2 = P * P, PIECES = BN / 8, ROWS = NT / PIECES;      // tokens the workgroup stores at a time
    constexpr int GROUPS = ROWS > P2 ? ROWS / P2 : 1, TOK = ROWS > P2 ? 1 : P2 / ROWS;   // patches at a time; tokens of a lane
    const int lw = LP - p.mw;                          // log2 of the pooled columns
    const int cc = tid % PIECES, t0 = tid / PIECES % P2, g = tid / (PIECES * P2);
    int src[TOK], h[TOK], w[TOK];
    size_t dst[TOK];
#pragma unroll
    for (int k = 0; k < TOK; ++k) {
        const int tk = t0 + k * ROWS;
        h[k] = tk >> LP;
        w[k] = n0 + cc * 8 < p.N ? tk & (P - 1) : 0x7fffffff;
        src[k] = (((h[k] >> p.mh) << lw) + ((tk & (P - 1)) >> p.mw)) * (BN * 2) + cc * 16;
        dst[k] = ((size_t)h[k] * p.geom.Wt + (tk & (P - 1))) * p.N + n0 + cc * 8;
    }
    unsigned short *const out = reinterpret_cast<unsigned short *>(p.C);
    auto patches = [&](auto whole_lines) {
#pragma unroll 2
        for (int d = g; d < count; d += GROUPS) {
            const PatchAt a = at[d];
            u32x4_t v[TOK];
#pragma unroll
            for (int k = 0; k < TOK; ++k) v[k] = *reinterpret_cast<const u32x4_t *>(stg + d * nc * (BN * 2) + src[k]);
#pragma unroll
            for (int k = 0; k < TOK; ++k)
                if (h[k] < a.hv && w[k] < a.wv) {
                    u32x4_t *q = reinterpret_cast<u32x4_t *>(out + a.at + dst[k]);
                    if constexpr (whole_lines) __builtin_nontemporal_store(v[k], q);
                    else *q = v[k];
                }
        }
    };
    // Non-temporal stores where a token's piece is whole 128-byte lines; otherwise a line is written by two tiles, and
    // ordinary stores let the L2 put it together (680 channels: 59 -> 43 us a call, 408: 67 -> 46).
    if (p.N % 64 == 0) patches(std::true_type{});
    else patches(std::false_type{});
}

// Reverse projection of one tile held in LDS as fp32 ct[row][cts]; rows are (patch, basis).  A lane expands one (patch,
// channel pair) per pass to its pooled tokens; those go back to LDS, over the rows that the pass has read, and
// from there to memory with the code that all selections share.  (Storing the p^2 tokens from the lanes that
// computed them made 9 KB of straight code for each of 16 selections, fetched cold by every launch: of the 3.7 us from
// the last product to the last store of a one-image call 2.3 were spent before the first store; a tile's
// 16 patches of ViT-B fc1 took 6.2 us.)
template <int LP, int MH, int MW, int BN, int NT>
__device__ __forceinline__ void unproject_tile(float *ct, int cts, int zero_row, const Params &p, const PatchAt *at, int n0, int tid)
{
    constexpr int P = 1 << LP;
    constexpr int PWd = P >> MW;
    constexpr int NC = (P >> MH) * PWd;
    constexpr float scale = 1.0f / (float)(P * P);
    constexpr int HALF = BN / 2, PASS = NT / HALF;      // channel pairs of a tile; patches per pass
    const int patches = p.bm_step / p.r;
    const int slot = tid / HALF, cp = tid % HALF;
    for (int base = 0; base < patches; base += PASS) {
        const int pt = base + slot, here = min(PASS, patches - base);
        // patches whose pooled tokens fit the rows that have been read by then
        const int part = min(here, (base + here) * p.r * cts * 4 / (NC * BN * 2));
        uint32_t tok[NC];
        if (pt < patches) {
            const float *src = ct + (size_t)(pt * p.r) * cts + 2 * cp, *zero = ct + zero_row * cts + 2 * cp;
            float c0[NC], c1[NC];
#pragma unroll
            for (int j = 0; j < NC; ++j) {              // (the same for every lane; all reads in flight together)
                const float2 t = *reinterpret_cast<const float2 *>((p.sel.mask >> j) & 1u ? src + (int)p.sel.pos[j] * cts : zero);
                c0[j] = t.x;
                c1[j] = t.y;
            }
            fwht_inplace<NC>(c0);
            fwht_inplace<NC>(c1);
#pragma unroll
            for (int j = 0; j < NC; ++j) tok[j] = pack_bf16x2(c0[j] * scale, c1[j] * scale);
        }
        if (part == 0) {        // 4 wavefronts, one basis, 16 pooled tokens: no room, the lanes store their tokens themselves
            if constexpr (NC * BN * 2 > PASS * (BN + 8) * 4) {
                const PatchAt a = pt < patches ? at[pt] : PatchAt{0, 0, 0};
                if (n0 + 2 * cp < p.N) {
#pragma unroll
                    for (int j = 0; j < NC; ++j)
                        for (int d = 0; d < 1 << (MH + MW); ++d) {
                            const int h = (j / PWd << MH) + (d >> MW), w = (j % PWd << MW) + (d & ((1 << MW) - 1));
                            if (h < a.hv && w < a.wv)
                                reinterpret_cast<uint32_t *>(p.C)[(a.at + ((size_t)h * p.geom.Wt + w) * p.N + n0) / 2 + cp] = tok[j];
                        }
                }
            }
            continue;
        }
        __syncthreads();                                // the pass's rows have been read, and what an earlier pass staged
        unsigned char *stg = reinterpret_cast<unsigned char *>(ct);
        for (int d0 = 0; d0 < here; d0 += part) {
            if (slot >= d0 && slot < d0 + part && pt < patches) {
#pragma unroll
                for (int j = 0; j < NC; ++j)
                    *reinterpret_cast<uint32_t *>(stg + ((slot - d0) * NC + j) * (BN * 2) + cp * 4) = tok[j];
            }
            __syncthreads();
            store_pooled<LP, BN, NT>(stg, min(part, here - d0), NC, at + base + d0, p, n0, tid);
            if (d0 + part < here) __syncthreads();
        }
    }
}

// The same without a barrier: a patch is the job of one wavefront from its coefficients to its tokens in memory.  A lane reads the coefficients of a channel pair and expands them to the pooled tokens; those go back to LDS as
// bf16, over the patch's own rows, and from there to memory, 16 bytes a lane, four pooled tokens at a time, each to all
// tokens of its group.  Rows too few to hold all pooled tokens take them in turns.
// For products in slices that join inside a launch of one workgroup a unit: few tiles, whose last workgroup everybody waits for (one
// image 768 -> 3072 r = 8 16.5 -> 15.7 us a call).  Larger launches write memory as fast as it takes it, and 8 patches at a time in place of
// one make it slower (131072 tokens 768 -> 768 r = 16 186 -> 190 us, 8192 tokens 1024 -> 4096 r = 4 in slices 34.0 -> 34.4).
template <int LP, int MH, int MW, int BN, int NT, int ZERO_ROW>
__device__ __forceinline__ void unproject_patches(float *ct, const Params &p, const PatchAt *at, int n0)
{
    constexpr int P = 1 << LP, CTS = BN + 8;
    constexpr int PWd = P >> MW, NC = (P >> MH) * PWd, COPIES = 1 << (MH + MW);
    constexpr float scale = 1.0f / (float)(P * P);
    constexpr int PIECES = BN / 8;              // of 16 bytes of a token
    static_assert(BN == 128, "a lane is a channel pair");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int patches = p.bm_step / p.r;
    const int piece = lane % PIECES, grp = lane / PIECES;      // grp: 0 to 3
    // pooled tokens that the patch's rows hold at a time (a power of two, at least 2)
    int fit = NC;
    while (fit * BN * 2 > p.r * CTS * 4) fit >>= 1;
    const int shift = __builtin_ctz(fit);
    unsigned short *const out = reinterpret_cast<unsigned short *>(p.C) + n0 + piece * 8;
    const bool whole_lines = p.N % 64 == 0, inside = n0 + piece * 8 < p.N;
    // Non-temporal stores where a token's piece is whole 128-byte lines; otherwise a line is written by two tiles, and
    // ordinary stores let the L2 put it together (680 channels: 59 -> 43 us a call, 408: 67 -> 46).
    auto put = [&](u32x4_t v, unsigned short *q) {
        if (whole_lines) __builtin_nontemporal_store(v, reinterpret_cast<u32x4_t *>(q));
        else *reinterpret_cast<u32x4_t *>(q) = v;
    };
    const size_t row = (size_t)p.geom.Wt * p.N;
    constexpr int QUADS = NC >= 4 ? NC / 4 : 1;
    size_t first_token[QUADS];      // element offset of pooled token 4 * quad + grp in its patch
#pragma unroll
    for (int kk = 0; kk < QUADS; ++kk) first_token[kk] = ((kk * 4 + grp) / PWd << MH) * row + (size_t)((kk * 4 + grp) % PWd << MW) * p.N;
    for (int pt = wave; pt < patches; pt += NT / 64) {
        const PatchAt a = at[pt];
        if (a.hv == 0) break;                       // (behind the last patch lie rows of tokens outside the grid)
        const float *const src = ct + (size_t)(pt * p.r) * CTS + 2 * lane, *const zero = ct + ZERO_ROW * CTS + 2 * lane;
        float c0[NC], c1[NC];
#pragma unroll
        for (int j = 0; j < NC; ++j) {              // (the same for every lane; all reads in flight together)
            const float2 t = *reinterpret_cast<const float2 *>((p.sel.mask >> j) & 1u ? src + (int)p.sel.pos[j] * CTS : zero);
            c0[j] = t.x;
            c1[j] = t.y;
        }
        fwht_inplace<NC>(c0);
        fwht_inplace<NC>(c1);
        uint32_t tok[NC];
#pragma unroll
        for (int j = 0; j < NC; ++j) tok[j] = pack_bf16x2(c0[j] * scale, c1[j] * scale);
        unsigned char *const stg = reinterpret_cast<unsigned char *>(ct + (size_t)(pt * p.r) * CTS);
        const int wv = inside ? a.wv : 0;
        if (NC >= 4 && fit == NC) {
            // (a wavefront's LDS operations are carried out in order)
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int j = 0; j < NC; ++j) *reinterpret_cast<uint32_t *>(stg + j * (BN * 2) + lane * 4) = tok[j];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            u32x4_t v[QUADS];
#pragma unroll
            for (int kk = 0; kk < QUADS; ++kk) v[kk] = *reinterpret_cast<const u32x4_t *>(stg + (kk * 4 + grp) * (BN * 2) + piece * 16);
            unsigned short *const to = out + a.at;
            if (a.hv >= P && wv >= P) {
#pragma unroll
                for (int kk = 0; kk < QUADS; ++kk)
#pragma unroll
                    for (int copy = 0; copy < COPIES; ++copy) put(v[kk], to + first_token[kk] + (copy >> MW) * row + (size_t)(copy & ((1 << MW) - 1)) * p.N);
            } else {
                for (int copy = 0; copy < COPIES; ++copy)
#pragma unroll
                    for (int kk = 0; kk < QUADS; ++kk) {
                        const int dh = copy >> MW, dw = copy & ((1 << MW) - 1);
                        if (((kk * 4 + grp) / PWd << MH) + dh < a.hv && ((kk * 4 + grp) % PWd << MW) + dw < wv)
                            put(v[kk], to + first_token[kk] + dh * row + (size_t)dw * p.N);
                    }
            }
            continue;
        }
        for (int first = 0; first < NC; first += fit) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int j = 0; j < NC; ++j)
                if (j >= first && j < first + fit) *reinterpret_cast<uint32_t *>(stg + (j - first) * (BN * 2) + lane * 4) = tok[j];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (NC >= 4 && fit >= 4) {
                for (int quad = 0; quad < fit; quad += 4) {
                    const int j = first + quad + grp, h = j / PWd << MH, w = j % PWd << MW;
                    const u32x4_t v = *reinterpret_cast<const u32x4_t *>(stg + (quad + grp) * (BN * 2) + piece * 16);
                    unsigned short *const to = out + a.at + h * row + (size_t)w * p.N;
#pragma unroll
                    for (int copy = 0; copy < COPIES; ++copy) {
                        const int dh = copy >> MW, dw = copy & ((1 << MW) - 1);
                        if (h + dh < a.hv && w + dw < wv) put(v, to + dh * row + (size_t)dw * p.N);
                    }
                }
                continue;
            }
            const int steps = fit * COPIES >> 2;
            for (int k = 0; k < (steps > 0 ? steps : 1); ++k) {
                const int n = k * 4 + grp, local = n & (fit - 1), j = first + local, copy = n >> shift;
                const int h = (j / PWd << MH) + (copy >> MW), w = ((j % PWd) << MW) + (copy & ((1 << MW) - 1));
                const u32x4_t v = *reinterpret_cast<const u32x4_t *>(stg + local * (BN * 2) + piece * 16);
                if (copy < COPIES && h < a.hv && w < wv) put(v, out + a.at + h * row + (size_t)w * p.N);
            }
        }
    }
}

// Eight entries of the sign matrix over 64, token `token` and bases 8 * piece ..., as bf16; zero past the last basis.
__device__ __forceinline__ uint4 sign_piece(const Params &p, int piece, int token)
{
    piece = __builtin_amdgcn_readfirstlane(piece);
    uint32_t v[4];
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
        const int k = piece * 8 + e;
        const uint32_t lo = k < p.r ? 0x3c80u | (unsigned)(__popc(p.nat[k] & token) & 1) << 15 : 0u;
        const uint32_t hi = k + 1 < p.r ? 0x3c80u | (unsigned)(__popc(p.nat[k + 1] & token) & 1) << 15 : 0u;
        v[e / 2] = lo | hi << 16;
    }
    return make_uint4(v[0], v[1], v[2], v[3]);
}

// Rows [lo, hi) of the tile that belong to tokens outside the grid (global row >= Q*r): empty
// for all but the last tiles.
__device__ __forceinline__ void extra_row_range(const Params &p, int m0, int &lo, int &hi)
{
    const long first = p.Q * p.r;
    const long l = first - m0, h = (long)p.M - m0;
    lo = l < 0 ? 0 : (int)(l < p.bm_step ? l : p.bm_step);
    hi = (int)(h < p.bm_step ? h : p.bm_step);
}

// A ring of `stages` LDS stages, each `depth` (32 or 64) elements of the reduction deep, as one number (a template parameter);
// whole: fragments are read a whole stage ahead.
constexpr int ring(int stages, int depth, bool whole = false) { return (whole ? 4096 : 0) + depth * 16 + stages; }
constexpr int ring_stages(int r) { return r % 16; }
constexpr int ring_depth(int r) { return r % 4096 / 16; }
constexpr bool ring_whole(int r) { return r >= 4096; }

// LDS layout of one stage.  A wavefront's load fills 1 KB of LDS in lane order, so rows cannot be padded; what a lane
// fetches is permuted instead.  Half a wavefront's transposing read touches 32 bytes each of rows k to k + 3 and k + 8 to
// k + 11 of a reduction-slow operand: 64-byte pieces are exchanged, xor k % 4, and 32-byte pieces, xor k / 8 % 2, so that
// the eight fall into different banks (rows of 128 and 384 bytes start in alternate halves of the banks by themselves: xor
// k / 2 % 2 for the 64-byte pieces).
// Reduction-fast rows of 128 or 64 bytes: 16-byte pieces, xor with a half or a quarter of the row number.
// (16 lanes of a read are rows 0 to 3 and 12 to 15 of one piece and 4 to 11 of its neighbour, which meet in the same banks in rows of 64
// bytes: 11 % of a unit's cycles in the exact input gradient.  Xor with 0, 2, 3, 1 for the quarters has no conflicts and changes nothing:
// both exact products of 16384 tokens 768 -> 3072 151.8 and 151.9 us.)
template <int BM, int BN, bool A_KFAST, int RING_OF>
struct Smem {
    static constexpr int DEPTH = ring_depth(RING_OF), STAGES = ring_stages(RING_OF);
    static constexpr int SA = A_KFAST ? DEPTH * 2 : BM * 2, SB = BN * 2;
    static constexpr int A_BYTES = BM * DEPTH * 2, B_BYTES = BN * DEPTH * 2;
    static constexpr int STAGE = A_BYTES + B_BYTES;
    static constexpr int RING = STAGES * STAGE;
    template <int ROW> __device__ static constexpr int swizzle(int k)       // of a reduction-slow row of ROW elements, in bytes
    {
        return (ROW % 128 == 0 ? (k & 3) << 6 : ((k >> 1) & 1) << 6) | ((k >> 3) & 1) << 5;
    }
    __device__ static constexpr int fast_swizzle(int row)                   // of a reduction-fast row, in pieces
    {
        return DEPTH == 64 ? (row >> 1) & 7 : (row >> 2) & 3;
    }
};

// 16 bytes a lane from `base` + `offset` to 1 KB of LDS at byte address `lds` (base and lds the same for the whole wavefront).  In
// assembly, so that the compiler does not wait for every such load in front of every LDS read: the main loop places the waits.
// (M0 is a reserved register: the compiler sets it right before a use of its own and keeps nothing in it.)
__device__ __forceinline__ void load_to_lds(const void *base, unsigned offset, unsigned lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(offset), "s"(base));
}

// All but the newest `LOADS` loads of this wavefront have arrived.
template <int LOADS>
__device__ __forceinline__ void loads_arrived()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LOADS) : "memory");
}

// Main loop of one tile on a ring of LDS stages; adds to acc.  `meanwhile` is called while the first loads are on
// their way.
template <int BM, int BN, int WGM, int WGN, int RING_OF, bool A_KFAST, int TM, int TN, typename F>
__device__ __forceinline__ void main_loop(const Plain &p, int m0, int n0, int kbeg, int kend, unsigned char *smem,
                                                acc_t (&acc)[TM][TN], F &&meanwhile)
{
    using S = Smem<BM, BN, A_KFAST, RING_OF>;
    constexpr int NT = 64 * WGM * WGN, WAVES = WGM * WGN;
    constexpr int WM = BM / WGM, WN = BN / WGN;
    constexpr int DEPTH = S::DEPTH, STAGES = S::STAGES, SUBS = DEPTH / 32;
    constexpr int SA = S::SA, SB = S::SB, A_BYTES = S::A_BYTES, STAGE = S::STAGE;
    // A stage is A's pieces of 16 bytes, then B's; a wavefront fetches 64 of them, 1 KB, at a time, and the first MORE wavefronts
    // may do so once more than the others.
    constexpr int A_KB = BM * DEPTH / 512, B_KB = BN * DEPTH / 512, LOADS = (A_KB + B_KB + WAVES - 1) / WAVES, MORE = (A_KB + B_KB) % WAVES;
    static_assert(BM * DEPTH % 512 == 0 && BN * DEPTH % 512 == 0, "a wavefront's load is of one operand");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WGN, wn = wave - wm * WGN;

    // what this lane fetches: byte offsets from the stage's first row (A reduction-fast: from row m0, at the stage's first k)
    constexpr int FAST = DEPTH / 8;             // pieces of a reduction-fast row
    const unsigned short *const abase = p.A + (A_KFAST ? (size_t)m0 * p.lda : 0), *const bbase = p.B;
    auto fetches_a = [&](int i) { return (i + 1) * WAVES <= A_KB || (i * WAVES < A_KB && wave < A_KB - i * WAVES); };
    auto fetches = [&](int i) { return MORE == 0 || i + 1 < LOADS || wave < MORE; };
    unsigned off[LOADS];
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
        if (fetches_a(i)) {
            const int c = tid + i * NT;
            if (A_KFAST) {
                const int row = c / FAST, piece = (c % FAST) ^ S::fast_swizzle(row);
                off[i] = (unsigned)(min(row, p.M - 1 - m0) * p.lda + piece * 8) * 2u;
            } else {
                const int k = c / (BM / 8), cc = (c - k * (BM / 8)) ^ (S::template swizzle<BM>(k) >> 4);
                off[i] = (unsigned)(k * p.lda + min(m0 + cc * 8, p.M - 8)) * 2u;
            }
        } else {
            const int c = tid + i * NT - A_KB * 64;
            const int k = c / (BN / 8), cc = (c - k * (BN / 8)) ^ (S::template swizzle<BN>(k) >> 4);
            off[i] = (unsigned)(k * p.ldb + min(n0 + cc * 8, p.N - 8)) * 2u;
        }
    }
    const unsigned lds0 = (unsigned)(size_t)LBP_LDS_PTR(unsigned char, smem) + wave * 1024;
    auto fetch_one = [&](int i, int k0, unsigned stage) {
        const unsigned short *a = abase + (A_KFAST ? (size_t)k0 : (size_t)k0 * p.lda), *b = bbase + (size_t)k0 * p.ldb;
        if (fetches(i)) load_to_lds(fetches_a(i) ? a : b, off[i], lds0 + stage + i * (WAVES * 1024));
    };
    auto fetch = [&](int s, unsigned stage, int first, int last) {
#pragma unroll
        for (int i = 0; i < LOADS; ++i)
            if (i >= first && i < last) fetch_one(i, kbeg + s * DEPTH, stage);
    };
    // All but the newest NEWER stages have arrived, and this wavefront's LDS reads, and so for every wavefront.
    auto arrive_and_sync = [&](auto newer) {
        constexpr int NEWER = decltype(newer)::value;
        __builtin_amdgcn_sched_barrier(0);
        if (MORE == 0 || NEWER == 0 || wave < MORE) loads_arrived<NEWER * LOADS>();
        else loads_arrived<NEWER *(LOADS - 1)>();
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };

    const int grp = lane >> 4, i16 = lane & 15, kr = 8 * grp + (i16 >> 2);
    int a_off[TM][2], b_off[TN][2];
#pragma unroll
    for (int mi = 0; mi < TM; ++mi)
#pragma unroll
        for (int h = 0; h < 2; ++h)
            a_off[mi][h] = A_KFAST ? (wm * WM + mi * 32 + h * 16 + i16) * SA
                                   : kr * SA + (((wm * WM + mi * 32 + h * 16 + 4 * (i16 & 3)) * 2) ^ S::template swizzle<BM>(kr));
#pragma unroll
    for (int ni = 0; ni < TN; ++ni)
#pragma unroll
        for (int h = 0; h < 2; ++h)
            b_off[ni][h] = A_BYTES + kr * SB + (((wn * WN + ni * 32 + h * 16 + 4 * (i16 & 3)) * 2) ^ S::template swizzle<BN>(kr));
    auto transposed = [](const unsigned char *q, int pitch) {      // the lane's 8 k-values of its column
        i16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LBP_LDS_PTR(i16x4_t, q));
        i16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LBP_LDS_PTR(i16x4_t, q + 4 * pitch));
        return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    // WHOLE: registers hold two stages' fragments, one being multiplied, the next being read.  Otherwise a stage is taken in
    // parts, and they hold two of those: sub-steps, or halves of A's rows in them where registers or (two stages) the time in front
    // of the barrier are short.
    constexpr bool WHOLE = ring_whole(RING_OF);
    constexpr int HALVES = !WHOLE && (TM > 2 || (TM == 2 && (STAGES == 2 || SUBS == 1))) ? 2 : 1, TA = TM / HALVES, PARTS = SUBS * HALVES;
    static_assert(WHOLE || PARTS % 2 == 0, "parts alternate between two sets of registers");
    constexpr bool B_LATER = BM * BN <= 128 * 128;
    constexpr int A_LOADS = A_KB / WAVES;
    auto one_a = [&](const unsigned char *s, int ks, int mi, int h) {
        const unsigned char *q = s + a_off[mi][h];
        return A_KFAST ? *reinterpret_cast<const bf16x8_t *>(q + (((ks * 4 + grp) ^ S::fast_swizzle(i16)) << 4)) : transposed(q + ks * 32 * SA, SA);
    };
    auto load_a = [&](const unsigned char *s, int ks, int half, bf16x8_t (&a)[TA][2]) {
#pragma unroll
        for (int mi = 0; mi < TA; ++mi)
#pragma unroll
            for (int h = 0; h < 2; ++h) a[mi][h] = one_a(s, ks, half * TA + mi, h);
    };
    auto load_b = [&](const unsigned char *s, int ks, bf16x8_t (&b)[TN][2]) {
#pragma unroll
        for (int ni = 0; ni < TN; ++ni)
#pragma unroll
            for (int h = 0; h < 2; ++h) b[ni][h] = transposed(s + b_off[ni][h] + ks * 32 * SB, SB);
    };
    auto product = [&](int half, const bf16x8_t (&a)[TA][2], const bf16x8_t (&b)[TN][2]) {
#pragma unroll
        for (int mi = 0; mi < TA; ++mi)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int ni = 0; ni < TN; ++ni)
#pragma unroll
                    for (int w = 0; w < 2; ++w) {
                        f32x4_t &c = acc[half * TA + mi][ni][2 * h + w];
                        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[ni][w], a[mi][h], c, 0, 0, 0);
                    }
    };
    constexpr int READS_A = 2 * TA * (A_KFAST ? 1 : 2), READS = READS_A + TN * 4, MFMAS = 4 * TA * TN;
    const int nfull = (kend - kbeg) / DEPTH;
    if (nfull > 0) {
#pragma unroll
        for (int j = 0; j < STAGES; ++j)
            if (j < nfull) fetch(j, j * STAGE, 0, LOADS);
        meanwhile();
        // `newer` stages that may still be on their way; STAGES - 2 in the loop, fewer behind the last request
        auto stage_and_sync = [&](int newer) {
            if (newer >= STAGES - 2) arrive_and_sync(std::integral_constant<int, STAGES - 2>{});
            else if (STAGES > 3 && newer == STAGES - 3) arrive_and_sync(std::integral_constant<int, (STAGES > 3 ? STAGES - 3 : 0)>{});
            else if (STAGES > 4 && newer == STAGES - 4) arrive_and_sync(std::integral_constant<int, (STAGES > 4 ? STAGES - 4 : 0)>{});
            else arrive_and_sync(std::integral_constant<int, 0>{});
        };
        if (nfull >= STAGES) arrive_and_sync(std::integral_constant<int, STAGES - 1>{});
        else stage_and_sync(nfull - 1);
        unsigned cur = 0;                       // LDS stage of step s
        auto next = [&]() { cur = cur + STAGE < (unsigned)S::RING ? cur + STAGE : 0; };
        if constexpr (WHOLE) {
            bf16x8_t a[2][SUBS][TA][2], b[2][SUBS][TN][2];
            auto read = [&](int set, int ks) {
                load_b(smem + cur, ks, b[set][ks]);
                load_a(smem + cur, ks, 0, a[set][ks]);
            };
#pragma unroll
            for (int ks = 0; ks < SUBS; ++ks) read(0, ks);
            // fragment n of a stage, in the order in which they are multiplied: of a sub-step, B's, then A's
            constexpr int READS_N = 2 * (TM + TN);
            auto read_n = [&](int set, int n) {
                const int ks = n / READS_N, f = n - ks * READS_N;
                if (f < 2 * TN) b[set][ks][f >> 1][f & 1] = transposed(smem + cur + b_off[f >> 1][f & 1] + ks * 32 * SB, SB);
                else a[set][ks][(f - 2 * TN) >> 1][f & 1] = one_a(smem + cur, ks, (f - 2 * TN) >> 1, f & 1);
            };
            auto mfma_n = [&](int set, int n) {
                const int ks = n / MFMAS, f = n - ks * MFMAS, mh = f / (2 * TN), nw = f - mh * 2 * TN;
                f32x4_t &c = acc[mh >> 1][nw >> 1][2 * (mh & 1) + (nw & 1)];
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[set][ks][nw >> 1][nw & 1], a[set][ks][mh >> 1][mh & 1], c, 0, 0, 0);
            };
            // one step: behind the barrier nobody reads stage s any more and the next one is complete
            auto step = [&](int s, auto set_, auto steady_) {
                constexpr int set = decltype(set_)::value;
                constexpr bool steady = decltype(steady_)::value;
                const unsigned freed = cur;
                if constexpr (steady) arrive_and_sync(std::integral_constant<int, STAGES - 2>{});
                else stage_and_sync(nfull - 2 - s);
                next();
                // the matrix instructions in LOADS groups, a load behind each
                constexpr int ALL = MFMAS * SUBS, RD = READS_N * SUBS;
#pragma unroll
                for (int g = 0; g < LOADS; ++g) {
#pragma unroll
                    for (int n = g * RD / LOADS; n < (g + 1) * RD / LOADS; ++n) read_n(set ^ 1, n);
#pragma unroll
                    for (int n = g * ALL / LOADS; n < (g + 1) * ALL / LOADS; ++n) mfma_n(set, n);
                    interleave_mfma_with_lds_reads<0, ALL / LOADS, (READS * SUBS + LOADS - 1) / LOADS>();
                    __builtin_amdgcn_sched_barrier(0);
                    if (steady || s + STAGES < nfull) fetch_one(g, kbeg + (s + STAGES) * DEPTH, freed);
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            int s = 0;
            for (; s + STAGES + 1 < nfull; s += 2) {
                step(s, std::integral_constant<int, 0>{}, std::true_type{});
                step(s + 1, std::integral_constant<int, 1>{}, std::true_type{});
            }
            for (; s + 2 < nfull; s += 2) {
                step(s, std::integral_constant<int, 0>{}, std::false_type{});
                step(s + 1, std::integral_constant<int, 1>{}, std::false_type{});
            }
            if (s + 1 < nfull) {
                step(s, std::integral_constant<int, 0>{}, std::false_type{});
#pragma unroll
                for (int ks = 0; ks < SUBS; ++ks) {
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
#pragma unroll
                        for (int mi = 0; mi < TA; ++mi) a[0][ks][mi][h] = a[1][ks][mi][h];
#pragma unroll
                        for (int ni = 0; ni < TN; ++ni) b[0][ks][ni][h] = b[1][ks][ni][h];
                    }
                }
            }
#pragma unroll
            for (int ks = 0; ks < SUBS; ++ks) product(0, a[0][ks], b[0][ks]);
        } else {
            bf16x8_t a[2][TA][2], b[2][TN][2];
            load_a(smem, 0, 0, a[0]);
            load_b(smem, 0, b[0]);
            unsigned freed = 0;
            int b_stage = -1;
            auto step = [&](int s, auto set_, auto steady_) {
                constexpr int first = decltype(set_)::value;        // b's set of the step's first sub-step
                constexpr bool steady = decltype(steady_)::value;
                if (B_LATER && b_stage >= 0) fetch(b_stage, freed, A_LOADS, LOADS);
#pragma unroll
                for (int part = 0; part + 1 < PARTS; ++part) {
                    const int ks = part / HALVES, nks = (part + 1) / HALVES;
                    if (nks != ks) load_b(smem + cur, nks, b[(first + nks) & 1]);
                    load_a(smem + cur, nks, (part + 1) % HALVES, a[(part + 1) & 1]);
                    product(part % HALVES, a[part & 1], b[(first + ks) & 1]);
                    if (nks != ks) interleave_mfma_with_lds_reads<0, MFMAS, READS>();
                    else interleave_mfma_with_lds_reads<0, MFMAS, READS_A>();
                }
                freed = cur;
                if constexpr (steady) arrive_and_sync(std::integral_constant<int, STAGES - 2>{});
                else stage_and_sync(nfull - 2 - s);
                next();
                b_stage = steady || s + STAGES < nfull ? s + STAGES : -1;
                if (b_stage >= 0) fetch(b_stage, freed, 0, B_LATER ? A_LOADS : LOADS);
                load_b(smem + cur, 0, b[(first + SUBS) & 1]);
                load_a(smem + cur, 0, 0, a[0]);
                product(HALVES - 1, a[1], b[(first + SUBS - 1) & 1]);
                interleave_mfma_with_lds_reads<0, MFMAS, READS>();
            };
            int s = 0;
            if constexpr (SUBS == 2) {
                for (; s + STAGES < nfull; ++s) step(s, std::integral_constant<int, 0>{}, std::true_type{});
                for (; s + 1 < nfull; ++s) step(s, std::integral_constant<int, 0>{}, std::false_type{});
            } else {
                for (; s + STAGES + 1 < nfull; s += 2) {
                    step(s, std::integral_constant<int, 0>{}, std::true_type{});
                    step(s + 1, std::integral_constant<int, 1>{}, std::true_type{});
                }
                for (; s + 2 < nfull; s += 2) {
                    step(s, std::integral_constant<int, 0>{}, std::false_type{});
                    step(s + 1, std::integral_constant<int, 1>{}, std::false_type{});
                }
                if (s + 1 < nfull) {
                    step(s, std::integral_constant<int, 0>{}, std::false_type{});
#pragma unroll
                    for (int ni = 0; ni < TN; ++ni)
#pragma unroll
                        for (int h = 0; h < 2; ++h) b[0][ni][h] = b[1][ni][h];
                }
            }
#pragma unroll
            for (int part = 0; part < PARTS; ++part) {
                const int ks = part / HALVES, nks = (part + 1) / HALVES;
                if (part + 1 < PARTS) {
                    if (nks != ks) load_b(smem + cur, nks, b[nks & 1]);
                    load_a(smem + cur, nks, (part + 1) % HALVES, a[(part + 1) & 1]);
                }
                product(part % HALVES, a[part & 1], b[ks & 1]);
            }
        }
        __syncthreads();
    } else {
        meanwhile();
    }
    const int k0 = kbeg + nfull * DEPTH;
    if (k0 < kend) {                            // the partial step: zeros from kend on, through registers
        const unsigned short *a = abase + (A_KFAST ? (size_t)k0 : (size_t)k0 * p.lda), *b = bbase + (size_t)k0 * p.ldb;
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            if (!fetches(i)) break;
            const int c = tid + i * NT;
            const bool of_a = fetches_a(i);
            const int k = of_a ? (A_KFAST ? ((c % FAST) ^ S::fast_swizzle(c / FAST)) * 8 : c / (BM / 8)) : (c - A_KB * 64) / (BN / 8);
            uint4 v = make_uint4(0u, 0u, 0u, 0u);
            if (k0 + k < kend) v = *reinterpret_cast<const uint4 *>(reinterpret_cast<const unsigned char *>(of_a ? a : b) + off[i]);
            *reinterpret_cast<uint4 *>(smem + c * 16) = v;
        }
        __syncthreads();
#pragma unroll
        for (int ks = 0; ks < SUBS; ++ks) {
            bf16x8_t a[TA][2], b[TN][2];
            load_b(smem, ks, b);
#pragma unroll
            for (int half = 0; half < TM / TA; ++half) {
                load_a(smem, ks, half, a);
                product(half, a, b);
            }
        }
        __syncthreads();
    }
}

// LDS of the matrix-core epilogue (8 wavefronts): the tile's coefficients as bf16, the sign matrix, and the tokens that each
// wavefront is storing.
constexpr int kSignBytes = 64 * 128, kJobBytes = 32 * 128;

// Columns that a reverse projection in the epilogue takes at a time: wider tiles hand their accumulators over in turns, so that
// the rows of one turn fit what the ring leaves.
constexpr int epilogue_columns(int bn) { return bn > 128 ? 128 : bn; }

// Dynamic LDS of a workgroup: the ring, and what the epilogue needs after it (fp32 rows for the pooled reverse projection).
template <int BM, int BN, bool A_KFAST, int RING, int EPI>
constexpr int lds_bytes()
{
    constexpr int EB = epilogue_columns(BN);
    const int ring = Smem<BM, BN, A_KFAST, RING>::RING;
    const int rows = EPI == EPI_UNPROJECT ? (BM + 1) * (EB + 8) * 4
                     : EPI == EPI_UNPROJECT_MFMA ? (BM + 16) * EB * 2 + kSignBytes + 8 * kJobBytes : 0;
    return ring > rows ? ring : rows;
}

// Wavefronts a SIMD that a kernel's registers have to leave room for: four where two workgroups of 8 wavefronts with 64 accumulators a lane are to
// share a unit, whose LDS holds two of lds_bytes; 1, which asks for nothing, elsewhere (kernels with fewer accumulators leave as many by themselves, and
// the other tiles of 64 fill the LDS with one).
constexpr int min_waves(int bm, int bn, int lds) { return bm * bn == 128 * 256 && 2 * lds <= 160 * 1024 ? 4 : 1; }

// Split reductions that are combined inside the launch.  Every workgroup of a tile stores its partial
// accumulators, then counts itself in on the tile's counter; whichever comes last adds all the parts
// in slice order (so the sum does not depend on who came last) and goes on to the epilogue.  Nobody
// waits.  Parts travel from one XCD's L2 to another's: they are written and read with device-scope
// accesses (16 bytes a lane, sc1), which go to the point where the XCDs are coherent, so that no cache has
// to be written back or invalidated as a whole, which is what a device-scope fence would cost
// (measured: tens of microseconds per launch).  The last workgroup leaves the counter at zero.
// `rows`: 32-row blocks of this wavefront that hold rows of the matrix; the others are neither stored nor read (one
// image of 4 patches fills half a 64-row tile).
constexpr int kDeviceScope = 16;                // cache policy sc1 of a buffer access
__device__ __forceinline__ __amdgpu_buffer_rsrc_t parts_of(float *p, size_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(p, 0, (int)bytes, 0x00027000);
}

template <int TM, int TN>
__device__ __forceinline__ void store_part(float *slot, const acc_t (&acc)[TM][TN], int rows)
{
    const __amdgpu_buffer_rsrc_t to = parts_of(slot, (size_t)TM * TN * 64 * blockDim.x);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        if (i >= rows) break;
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, acc[i][j][q]), to, threadIdx.x * 16,
                                                       ((i * TN + j) * 4 + q) * blockDim.x * 16, kDeviceScope);
    }
}

// Adds `splits` parts, FLY of them in flight together: with one at a time the eight parts of a one-image call took 3.7 us,
// a trip to memory each; four at a time, 8 bytes a lane, 2.5; eight, 16 bytes, 1.5.  Where there are fewer, the last one is read again, so
// a caller with at most half as many asks for half: both gradients of 8 images 768 -> 3072 r = 8 in 4 slices 20.4 -> 19.2 us, 16 images
// 384 -> 1536 in 2 18.4 -> 17.4, 5 to 8 slices level (0 to 0.1 us; reads under a condition instead take 0.1 to 0.3 more with 3, 4 and 8).
template <int FLY, int TM, int TN>
__device__ __forceinline__ void add_parts(float *slots, size_t pitch, int splits, acc_t (&sum)[TM][TN], int rows)
{
    constexpr int NV = TN * 4;
    const __amdgpu_buffer_rsrc_t from = parts_of(slots, pitch * splits * sizeof(float));
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        if (i >= rows) break;
        for (int z = 0; z < splits; z += FLY) {
            f32x4_t v[FLY][NV];
#pragma unroll
            for (int f = 0; f < FLY; ++f)
#pragma unroll
                for (int q = 0; q < NV; ++q)
                    v[f][q] = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(
                        from, threadIdx.x * 16, (int)(min(z + f, splits - 1) * pitch * 4) + (i * NV + q) * (int)blockDim.x * 16, kDeviceScope));
            __builtin_amdgcn_sched_barrier(0);      // (all of them on their way before the first is waited for)
#pragma unroll
            for (int f = 0; f < FLY; ++f) {
                if (z + f >= splits) break;
#pragma unroll
                for (int q = 0; q < NV; ++q) sum[i][q >> 2][q & 3] += v[f][q];
            }
        }
    }
}

// One workgroup's share of a product: number `id` of its tiles x slices; `smem` is the workgroup's dynamic LDS
// (lds_bytes<BM, BN, A_KFAST, RING, EPI>() of them).
template <int BM, int BN, int WGM, int WGN, int RING, bool A_KFAST, int EPI, int LP, bool JOIN = false>
__device__ __forceinline__ void gemm_body(const ParamsOf<EPI> &p, const int id, unsigned char *smem)
{
    constexpr int NT = 64 * WGM * WGN;
    constexpr int WM = BM / WGM, WN = BN / WGN;
    constexpr int TM = WM / 32, TN = WN / 32;
    static_assert(WM % 32 == 0 && WN % 32 == 0, "wave tile must be made of 32x32 tiles");
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WGN, wn = wave - wm * WGN;

    // XCD-aware numbering: workgroup ids go round-robin over the 8 XCDs, each of which has an L2 of its own.  The XCDs form
    // xcd_s groups, every group taking each xcd_s-th slice of the reduction; in a group the tiles of one XCD form an
    // xcd_a x xcd_b block of the output, so that they share xcd_a strips of A and xcd_b strips of B (chosen on the host to
    // make what an XCD reads smallest)
    int tm, tn, slice;
    if (p.xcd_a > 0) {
        const int x = id & 7, i = id >> 3, per = p.xcd_a * p.xcd_b;
        const int xg = x / p.xcd_s, z = i / per, t = i - z * per;
        slice = z * p.xcd_s + (x - xg * p.xcd_s);
        const int bn = p.tiles_n / p.xcd_b;           // blocks along n
        const int xm = xg / bn, xn = xg - xm * bn;
        const int im = t / p.xcd_b, in = t - im * p.xcd_b;
        tm = xm * p.xcd_a + im;
        tn = xn * p.xcd_b + in;
    } else {                                          // a run of workgroups per XCD
        const int T = p.tiles_m * p.tiles_n * p.xcd_s, x = id & 7;
        const int at = x * (p.count >> 3) + min(x, p.count & 7) + (id >> 3);
        const int z = at / T, in_z = at - z * T, t = in_z / p.xcd_s;
        slice = z * p.xcd_s + (in_z - t * p.xcd_s);
        const int band = t / (p.run_band * p.tiles_n), first = band * p.run_band;
        const int rows = min(p.run_band, p.tiles_m - first), in_band = t - first * p.tiles_n;
        tn = in_band / rows;
        tm = first + in_band - tn * rows;
    }
    const int m0 = tm * p.bm_step, n0 = tn * BN;
    const int kbeg = slice * p.k_per_split;
    const int kend = min(p.K, kbeg + p.k_per_split);

    const int li = lane & 31, kg = lane >> 5, grp = lane >> 4, i16 = lane & 15;
    acc_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[i][j][q] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    // what the epilogue can know beforehand
    [[maybe_unused]] PatchAt *at = nullptr;
    [[maybe_unused]] uint4 signs;
    if constexpr (EPI == EPI_UNPROJECT) {
        __shared__ PatchAt patch_at[BM];
        at = patch_at;
    }
    main_loop<BM, BN, WGM, WGN, RING, A_KFAST>(p, m0, n0, kbeg, kend, smem, acc, [&]() {
        if constexpr (EPI == EPI_UNPROJECT) locate_patches(p, m0, p.bm_step / p.r, at, tid);
        if constexpr (EPI == EPI_UNPROJECT_MFMA) signs = sign_piece(p, wave, lane);
    });

    if constexpr (JOIN) {
        if (p.splits > 1) {
            __shared__ unsigned arrived;
            const int tile_id = tm * p.tiles_n + tn;
            float *const tile_parts = p.parts + (size_t)tile_id * p.splits * (BM * BN);
            const int rows = (min(p.M - m0, p.bm_step) - wm * WM + 31) >> 5;       // (may be negative: none)
            store_part<TM, TN>(tile_parts + (size_t)slice * (BM * BN), acc, rows);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_s_waitcnt(0);        // every lane's part has arrived before the workgroup counts itself in
            __syncthreads();
            if (tid == 0)
                arrived = __hip_atomic_fetch_add(p.counters + (size_t)tile_id * kCounterPitch, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            if (arrived != (unsigned)(p.splits - 1)) return;      // the same for every lane of the workgroup
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q) acc[i][j][q] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            static_assert(TN == 1, "registers for four parts in flight");
            constexpr int FLY = ring_stages(RING) > 3 && TM == 1 ? 8 : 4;
            if (p.splits > FLY / 2) add_parts<FLY>(tile_parts, BM * BN, p.splits, acc, rows);
            else add_parts<FLY / 2>(tile_parts, BM * BN, p.splits, acc, rows);
            if (tid == 0) __hip_atomic_store(p.counters + (size_t)tile_id * kCounterPitch, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    // Two column halves as bf16: the lane groups trade pieces, and each lane has eight neighbouring columns, from
    // 8 * (grp / 2) + 16 * (grp % 2) on.
    [[maybe_unused]] const int col8 = 8 * (grp >> 1) + 16 * (grp & 1);
    [[maybe_unused]] auto eight_columns = [](const f32x4_t &l, const f32x4_t &r) {
        const auto x = __builtin_amdgcn_permlane16_swap(pack_bf16x2(l[0], l[1]), pack_bf16x2(r[0], r[1]), false, false);
        const auto y = __builtin_amdgcn_permlane16_swap(pack_bf16x2(l[2], l[3]), pack_bf16x2(r[2], r[3]), false, false);
        return make_uint4(x[0], y[0], x[1], y[1]);
    };
    // The reverse projection takes EB columns at a time: the wavefronts that own them hand them over, all work on them.
    constexpr int EB = epilogue_columns(BN), TURNS = BN / EB;
    static_assert(WGN % TURNS == 0, "a wavefront's columns belong to one turn");
    [[maybe_unused]] const int my_turn = wn / (WGN / TURNS), my_col = (wn - my_turn * (WGN / TURNS)) * WN;
    if constexpr (EPI == EPI_UNPROJECT_MFMA) {
        // Eq. 7 for selections that cannot be pooled (patch 8): per patch, tokens[64][BN] =
        // (1/64) * S[64][r] * coefficients[r][BN] with S the +-1 matrix, on the matrix cores.
        // The tile's rows (patch, basis) go to LDS as bf16 in the layout of a reduction-slow operand, S / 64 as one whose
        // reduction index is contiguous.  Then a wavefront has jobs of its own, 32 tokens x 64 channels of a patch each, and
        // shares nothing any more: products, tokens to its own LDS, from there 16 bytes a lane to memory.
        static_assert(EB == 128 && BN % EB == 0 && LP == 3 && NT == 512, "matrix-core epilogue: 128 channels at a time, patch 8, 8 wavefronts");
        constexpr int S_CO = EB * 2;            // pitch of the coefficient rows; pieces of 64 bytes exchanged, xor row % 4
        unsigned char *cot = smem, *sgn = smem + (BM + 16) * S_CO, *stg = sgn + kSignBytes + wave * kJobBytes;
        *reinterpret_cast<uint4 *>(sgn + lane * 128 + ((wave ^ ((lane >> 1) & 7)) << 4)) = signs;
        uint4 rounded[TM][TN][2];
#pragma unroll
        for (int mi = 0; mi < TM; ++mi)
#pragma unroll
            for (int ni = 0; ni < TN; ++ni)
#pragma unroll
                for (int h = 0; h < 2; ++h) rounded[mi][ni][h] = eight_columns(acc[mi][ni][2 * h], acc[mi][ni][2 * h + 1]);
        const int ksteps = (p.r + 15) >> 4, patches = p.bm_step / p.r;
        // the last step, where it is not full, reads rows of the next patch (or rows behind the tile that nobody wrote): they must
        // not reach the product even times a zero sign, or one that is not finite would turn this patch's tokens into NaN
        uint4 keep;
        {
            const int left = p.r - (ksteps - 1) * 16 - kg * 8;      // coefficients of that step in this lane's 8
            auto two = [&](int e) { return (left > e ? 0xffffu : 0u) | (left > e + 1 ? 0xffff0000u : 0u); };
            keep = make_uint4(two(0), two(2), two(4), two(6));
        }
#pragma unroll 1
        for (int turn = 0; turn < TURNS; ++turn) {
            const int n0t = n0 + turn * EB;
            if (TURNS > 1 && turn > 0) {
                if (n0t >= p.N) break;
                __syncthreads();                    // the columns before have been read
            }
            if (TURNS == 1 || my_turn == turn) {
#pragma unroll
                for (int mi = 0; mi < TM; ++mi)
#pragma unroll
                    for (int ni = 0; ni < TN; ++ni)
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            const int row = wm * WM + mi * 32 + h * 16 + i16, col = (my_col + ni * 32 + col8) * 2;
                            *reinterpret_cast<uint4 *>(cot + row * S_CO + (col ^ ((row & 3) << 6))) = rounded[mi][ni][h];
                        }
            }
            __syncthreads();
            for (int job = wave; job < patches * 4; job += 8) {
                const int pt = job >> 2, mt = (job >> 1) & 1, c0 = (job & 1) * 64;
                const long q = (long)(m0 / p.r) + pt;
                if (q >= p.Q) break;
                f32x16_t o[2];
#pragma unroll
                for (int c = 0; c < 2; ++c)
#pragma unroll
                    for (int e = 0; e < 16; ++e) o[c][e] = 0.f;
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) {
                    if (ks < ksteps) {
                        const int row = pt * p.r + ks * 16 + 8 * (grp >> 1) + (i16 >> 2);
                        const unsigned char *qd = cot + row * S_CO;
                        const bf16x8_t sg = *reinterpret_cast<const bf16x8_t *>(sgn + (mt * 32 + li) * 128 +
                                                                                  (((ks * 2 + kg) ^ ((li >> 1) & 7)) << 4));
#pragma unroll
                        for (int c = 0; c < 2; ++c) {
                            const int col = ((c0 + c * 32 + 16 * (grp & 1) + 4 * (i16 & 3)) * 2) ^ ((row & 3) << 6);
                            i16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LBP_LDS_PTR(i16x4_t, qd + col));
                            i16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LBP_LDS_PTR(i16x4_t, qd + 4 * S_CO + col));
                            uint4 b = __builtin_bit_cast(uint4, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                            if (ks == ksteps - 1) b = make_uint4(b.x & keep.x, b.y & keep.y, b.z & keep.z, b.w & keep.w);
                            // rows of the product = channels, columns = tokens
                            o[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, b), sg, o[c], 0, 0, 0);
                        }
                    }
                }
                long img;
                int a0, b0;
                p.geom.origin(q, img, a0, b0);
                unsigned short *dst = reinterpret_cast<unsigned short *>(p.C) + p.geom.token(img, a0, b0) * p.N + n0t + c0;
                const int hv = p.geom.Ht - a0, wv = p.geom.Wt - b0;     // tokens of the patch inside the grid
                // element 4*g4+e of o[c]: channel c0 + c*32 + 8*g4 + 4*kg + e, token mt*32 + li.  Token rows of 128 bytes, 16-byte
                // pieces exchanged, xor half the token's number.
#pragma unroll
                for (int c = 0; c < 2; ++c)
#pragma unroll
                    for (int g4 = 0; g4 < 4; ++g4)
                        *reinterpret_cast<uint2 *>(stg + li * 128 + (((c * 4 + g4) ^ ((li >> 1) & 7)) << 4) + kg * 8) =
                            make_uint2(pack_bf16x2(o[c][g4 * 4], o[c][g4 * 4 + 1]), pack_bf16x2(o[c][g4 * 4 + 2], o[c][g4 * 4 + 3]));
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");      // (a wavefront's LDS operations are carried out in order)
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int tl = i * 8 + (lane >> 3), cc = lane & 7, h = mt * 4 + i, w = lane >> 3;
                    const u32x4_t v = *reinterpret_cast<const u32x4_t *>(stg + tl * 128 + ((cc ^ ((tl >> 1) & 7)) << 4));
                    if (n0t + c0 + cc * 8 < p.N && h < hv && w < wv) {
                        u32x4_t *const to = reinterpret_cast<u32x4_t *>(dst + ((size_t)h * p.geom.Wt + w) * p.N + cc * 8);
                        if (p.N % 64 == 0) __builtin_nontemporal_store(v, to);      // (as in store_pooled: 1896 channels r = 17 120 -> 100 us)
                        else *to = v;
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
            if (p.extra_rows > 0) {       // tokens outside the grid: bf16 rows of the product times 1/64 (exact)
                int lo, hi;
                extra_row_range(p, m0, lo, hi);
                for (int it = tid; it < (hi - lo) * (EB / 8); it += NT) {
                    const int lr = lo + it / (EB / 8), cc = it % (EB / 8);
                    const int col = n0t + cc * 8;
                    if (col >= p.N) continue;
                    const long j = (long)m0 + lr - p.Q * p.r;
                    const long img = j / p.extra;
                    const int e = (int)(j - img * p.extra);
                    uint4 v = *reinterpret_cast<const uint4 *>(cot + lr * S_CO + ((cc * 16) ^ ((lr & 3) << 6)));
                    constexpr float inv = 1.0f / 64.0f;
                    v.x = pack_bf16x2(bf16_lo_to_f32(v.x) * inv, bf16_hi_to_f32(v.x) * inv);
                    v.y = pack_bf16x2(bf16_lo_to_f32(v.y) * inv, bf16_hi_to_f32(v.y) * inv);
                    v.z = pack_bf16x2(bf16_lo_to_f32(v.z) * inv, bf16_hi_to_f32(v.z) * inv);
                    v.w = pack_bf16x2(bf16_lo_to_f32(v.w) * inv, bf16_hi_to_f32(v.w) * inv);
                    *reinterpret_cast<uint4 *>(reinterpret_cast<unsigned short *>(p.C) + ((size_t)img * p.geom.img + e) * p.N + col) = v;
                }
            }
        }
    } else if constexpr (EPI == EPI_UNPROJECT) {
        static_assert(BN % EB == 0, "turns of the same columns");
        constexpr int CTS = EB + 8;
        float *ct = reinterpret_cast<float *>(smem);
        // the loop above ended with a barrier: nobody reads operands any more
#pragma unroll 1
        for (int turn = 0; turn < TURNS; ++turn) {
            const int n0t = n0 + turn * EB;
            if (TURNS > 1 && turn > 0) {
                if (n0t >= p.N) break;
                __syncthreads();                    // the columns before have been stored
            }
            if (TURNS == 1 || my_turn == turn) {
#pragma unroll
                for (int mi = 0; mi < TM; ++mi)
#pragma unroll
                    for (int ni = 0; ni < TN; ++ni)
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            *reinterpret_cast<f32x4_t *>(ct + (wm * WM + mi * 32 + (q >> 1) * 16 + i16) * CTS + my_col + ni * 32 + (q & 1) * 16 + grp * 4) =
                                acc[mi][ni][q];
            }
            if (tid < EB / 4) *reinterpret_cast<f32x4_t *>(ct + BM * CTS + tid * 4) = f32x4_t{0.f, 0.f, 0.f, 0.f};
            __syncthreads();
            if (p.extra_rows > 0) {       // tokens outside the grid: their rows are the gradient itself, scaled (first:
                                          // the expansion reuses the rows)
                int lo, hi;
                extra_row_range(p, m0, lo, hi);
                constexpr float inv = 1.0f / (float)((1 << LP) * (1 << LP));
                constexpr int HALF = EB / 2;
                for (int it = tid; it < (hi - lo) * HALF; it += NT) {
                    const int lr = lo + it / HALF, cp = it % HALF;
                    const int col = n0t + 2 * cp;
                    if (col >= p.N) continue;
                    const long j = (long)m0 + lr - p.Q * p.r;
                    const long img = j / p.extra;
                    const int e = (int)(j - img * p.extra);
                    uint32_t *dst = reinterpret_cast<uint32_t *>(p.C) + (((size_t)img * p.geom.img + e) * p.N + col) / 2;
                    *dst = pack_bf16x2(ct[lr * CTS + 2 * cp] * inv, ct[lr * CTS + 2 * cp + 1] * inv);
                }
            }
            switch (p.mh * 4 + p.mw) {
#define LBP_CASE(MH, MW)                                                                         \
    case MH * 4 + MW:                                                                            \
        if constexpr (MH <= LP && MW <= LP && ((1 << LP) >> MH) * ((1 << LP) >> MW) <= 16) {    \
            if constexpr (JOIN && ring_stages(RING) > 3) unproject_patches<LP, MH, MW, EB, NT, BM>(ct, p, at, n0t);          \
            else unproject_tile<LP, MH, MW, EB, NT>(ct, CTS, BM, p, at, n0t, tid);                  \
        }                                                                                        \
            break;
                LBP_CASE(0, 0) LBP_CASE(0, 1) LBP_CASE(0, 2) LBP_CASE(0, 3)
                LBP_CASE(1, 0) LBP_CASE(1, 1) LBP_CASE(1, 2) LBP_CASE(1, 3)
                LBP_CASE(2, 0) LBP_CASE(2, 1) LBP_CASE(2, 2) LBP_CASE(2, 3)
                LBP_CASE(3, 0) LBP_CASE(3, 1) LBP_CASE(3, 2) LBP_CASE(3, 3)
#undef LBP_CASE
                default: break;
            }
        }
    } else {
#pragma unroll
        for (int mi = 0; mi < TM; ++mi)
#pragma unroll
            for (int ni = 0; ni < TN; ++ni)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int row = m0 + wm * WM + mi * 32 + h * 16 + i16, col = n0 + wn * WN + ni * 32;
                    const f32x4_t l = acc[mi][ni][2 * h] * p.scale, r = acc[mi][ni][2 * h + 1] * p.scale;
                    if (EPI == EPI_F32 || (EPI == EPI_PLAIN && !p.store_bf16)) {
                        float *to = reinterpret_cast<float *>(p.C) + ((size_t)slice * p.M + row) * p.N + col + grp * 4;
                        if (row < p.M && col + grp * 4 < p.N) *reinterpret_cast<f32x4_t *>(to) = l;
                        if (row < p.M && col + 16 + grp * 4 < p.N) *reinterpret_cast<f32x4_t *>(to + 16) = r;
                    } else {
                        const uint4 v = eight_columns(l, r);
                        if (row < p.M && col + col8 < p.N)
                            *reinterpret_cast<uint4 *>(reinterpret_cast<unsigned short *>(p.C) + (size_t)row * p.N + col + col8) = v;
                    }
                }
    }
}

template <int BM, int BN, int WGM, int WGN, int RING, bool A_KFAST, int EPI, int LP, bool JOIN = false>
__global__ __launch_bounds__(64 * WGM * WGN, min_waves(BM, BN, lds_bytes<BM, BN, A_KFAST, RING, EPI>())) void gemm_kernel(ParamsOf<EPI> p)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    gemm_body<BM, BN, WGM, WGN, RING, A_KFAST, EPI, LP, JOIN>(p, blockIdx.x, smem);
}

template <int BM, int BN, int WGM, int WGN, int RING, bool A_KFAST, int EPI, int LP, bool JOIN = false>
hipError_t launch_one(const Params &p, int splits, hipStream_t stream)
{
    constexpr int LDS = lds_bytes<BM, BN, A_KFAST, RING, EPI>();
    const dim3 grid((unsigned)(p.tiles_m * p.tiles_n) * (unsigned)splits);
    return LBP_LAUNCH_KERNEL((gemm_kernel<BM, BN, WGM, WGN, RING, A_KFAST, EPI, LP, JOIN>), grid, 64 * WGM * WGN, LDS, stream,
                             static_cast<const ParamsOf<EPI> &>(p));
}

// Two independent products in one launch: workgroups [0, blocks_first) run `first`, the rest run
// `second`.  A low-rank product alone leaves
// compute units idle (a hundred-odd tiles on 256 units); launched together the two products of
// Algorithm 1 (the weight gradient and the input gradient only share the read-only g^y) fill them
// and save one launch gap.  Both bodies are the ones of the single-product kernels, so results are
// bit-identical to separate launches.
template <int EPI1>
struct PairParams {
    ParamsOf<EPI1> first;
    Plain second;
    int blocks_first, blocks_second;
    int second_leads;     // 1: the workgroups of `second` have the lower indices (are dispatched first)
};

// ... and the bias gradient's rows, which workgroups behind those of the products add up: they run on units that no product
// needs any more.  (A kernel of its own: one for both, with its arguments and a comparison in every launch, costs calls without a bias
// gradient 0.15 to 0.5 us: 64 images 768 -> 3072 r = 8 30.2 -> 30.7, one image 10.8 -> 10.95, 48 -> 192 6.75 -> 7.0.)
template <int EPI1>
struct PairBiasParams : PairParams<EPI1> {
    BiasSum bias;
};
template <int EPI1, bool BIAS> struct PairParamsFor { typedef PairParams<EPI1> type; };
template <int EPI1> struct PairParamsFor<EPI1, true> { typedef PairBiasParams<EPI1> type; };

template <int WGM, int WGN, int ST1, int BM1, int BN1, bool KF1, int EPI1, int LP1, int ST2, int BM2, int BN2, bool KF2,
          int EPI2, int LP2, bool JOIN1, bool BIAS>
__global__ __launch_bounds__(64 * WGM * WGN, min_waves(BM1, BN1, lds_bytes<BM1, BN1, KF1, ST1, EPI1>())) void gemm_pair_kernel(typename PairParamsFor<EPI1, BIAS>::type pp)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    if constexpr (BIAS) {
        const int block = (int)blockIdx.x - (pp.blocks_first + pp.blocks_second);
        if (block >= 0) {
            bias_sum_block<16 * WGM * WGN, true>(pp.bias, block, reinterpret_cast<float4 *>(smem));
            return;
        }
    }
    // (both orders keep a tile's workgroup index modulo 8, hence its XCD, a function of its tile id only)
    const int b = pp.second_leads ? (blockIdx.x < (unsigned)pp.blocks_second ? (int)blockIdx.x + pp.blocks_first
                                                                             : (int)blockIdx.x - pp.blocks_second)
                                  : (int)blockIdx.x;
    if (b < pp.blocks_first) {
        gemm_body<BM1, BN1, WGM, WGN, ST1, KF1, EPI1, LP1, JOIN1>(pp.first, b, smem);
    } else {
        gemm_body<BM2, BN2, WGM, WGN, ST2, KF2, EPI2, LP2>(pp.second, b - pp.blocks_first, smem);
    }
}

template <int WGM, int WGN, int ST1, int BM1, int BN1, bool KF1, int EPI1, int LP1, int ST2, int BM2, int BN2, bool KF2,
          int EPI2, int LP2, bool JOIN1 = false>
hipError_t launch_pair(const Params &first, int splits_first, const Params &second, int splits_second,
                       hipStream_t stream, bool second_leads, const BiasSum *bias)
{
    constexpr int L1 = lds_bytes<BM1, BN1, KF1, ST1, EPI1>(), L2 = lds_bytes<BM2, BN2, KF2, ST2, EPI2>();
    constexpr int LDS = L1 > L2 ? L1 : L2;
    PairBiasParams<EPI1> pp;
    pp.first = static_cast<const ParamsOf<EPI1> &>(first);
    pp.second = static_cast<const Plain &>(second);
    pp.blocks_first = first.tiles_m * first.tiles_n * splits_first;
    pp.blocks_second = second.tiles_m * second.tiles_n * splits_second;
    pp.second_leads = second_leads ? 1 : 0;
    const unsigned blocks = (unsigned)(pp.blocks_first + pp.blocks_second);
    if (bias) {
        pp.bias = *bias;
        return LBP_LAUNCH_KERNEL((gemm_pair_kernel<WGM, WGN, ST1, BM1, BN1, KF1, EPI1, LP1, ST2, BM2, BN2, KF2, EPI2, LP2, JOIN1, true>),
                                 dim3(blocks + bias->blocks), 64 * WGM * WGN, LDS, stream, pp);
    }
    return LBP_LAUNCH_KERNEL((gemm_pair_kernel<WGM, WGN, ST1, BM1, BN1, KF1, EPI1, LP1, ST2, BM2, BN2, KF2, EPI2, LP2, JOIN1, false>),
                             dim3(blocks), 64 * WGM * WGN, LDS, stream, static_cast<const PairParams<EPI1> &>(pp));
}

// All instantiations of one tile shape: output kind x operand layout; lp is
// log2(patch) for the fused reverse projection.  RING_X: the ring of input gradients without the pooled epilogue, where it is another.
template <int BM, int BN, int WGM, int WGN, int RING, bool FUSED, int RING_X = RING>
hipError_t launch_tile(const Params &p, bool a_kfast, GemmOut out, int lp, int splits, hipStream_t s)
{
    if (out == GemmOut::kUnproject) {
        if constexpr (FUSED) {
            if (p.splits > 1) {      // slices that join inside the launch: the 8-wavefront 128-wide tiles, patch 4 and 8
                if constexpr (BN == 128 && WGM * WGN == 8) {
                    if (lp == 2 && !p.mfma_epilogue) return launch_one<BM, BN, WGM, WGN, RING, true, EPI_UNPROJECT, 2, true>(p, p.splits, s);
                    if (lp != 3) return hipErrorInvalidValue;
                    if (p.mfma_epilogue) return launch_one<BM, BN, WGM, WGN, RING, true, EPI_UNPROJECT_MFMA, 3, true>(p, p.splits, s);
                    return launch_one<BM, BN, WGM, WGN, RING, true, EPI_UNPROJECT, 3, true>(p, p.splits, s);
                }
                return hipErrorInvalidValue;
            }
            if (p.mfma_epilogue) {
                if constexpr (BN % 128 == 0) {
                    if (lp == 3) return launch_one<BM, BN, WGM, WGN, RING_X, true, EPI_UNPROJECT_MFMA, 3>(p, 1, s);
                }
                return hipErrorInvalidValue;
            }
            if (lp == 3) return launch_one<BM, BN, WGM, WGN, RING, true, EPI_UNPROJECT, 3>(p, 1, s);
            if (lp == 2) return launch_one<BM, BN, WGM, WGN, RING, true, EPI_UNPROJECT, 2>(p, 1, s);
        }
        return hipErrorInvalidValue;
    }
    if (out == GemmOut::kF32) {
        if (a_kfast) return launch_one<BM, BN, WGM, WGN, RING_X, true, EPI_F32, 0>(p, splits, s);
        return launch_one<BM, BN, WGM, WGN, RING, false, EPI_F32, 0>(p, splits, s);
    }
    if (a_kfast) return launch_one<BM, BN, WGM, WGN, RING_X, true, EPI_BF16, 0>(p, 1, s);
    return launch_one<BM, BN, WGM, WGN, RING, false, EPI_BF16, 0>(p, 1, s);
}

}  // namespace mfma

// One entry per tile shape, defined in gemm_mfma_<shape>.hip.  `deep`: the longer of the shape's rings, fewer workgroups per
// compute unit.
hipError_t mfma_tile_128x128(const mfma::Params &p, bool a_kfast, GemmOut out, int lp, int splits, bool deep, hipStream_t s);
hipError_t mfma_tile_64x128(const mfma::Params &p, bool a_kfast, GemmOut out, int lp, int splits, bool deep, hipStream_t s);
hipError_t mfma_tile_128x256(const mfma::Params &p, bool a_kfast, GemmOut out, int lp, int splits, bool deep, hipStream_t s);
hipError_t mfma_tile_256x256(const mfma::Params &p, bool a_kfast, GemmOut out, int lp, int splits, bool deep, hipStream_t s);
hipError_t mfma_tile_64x64(const mfma::Params &p, bool a_kfast, GemmOut out, int lp, int splits, bool deep, hipStream_t s);
hipError_t mfma_tile_256x192(const mfma::Params &p, bool a_kfast, GemmOut out, int lp, int splits, bool deep, hipStream_t s);
hipError_t mfma_tile_256x128(const mfma::Params &p, bool a_kfast, GemmOut out, int lp, int splits, bool deep, hipStream_t s);

// Grouped launch of the input-gradient product `x` (A reduction-fast; tile 128x128 or 64x128 with 8
// wavefronts: bm_x = 128 or 64; or 128x256 with the fused epilogue: bn_x = 256; out_x as in launch_gemm, kUnproject needs patch 4 or 8, lp_x = log2 of it) and the
// weight-gradient product `w` (A reduction-slow, 128x128 tile with 8 wavefronts, fp32 or bf16 store
// by w.store_bf16).  hipErrorInvalidValue for a combination that is not instantiated.
hipError_t mfma_pair_w8(const mfma::Params &x, int bm_x, int bn_x, GemmOut out_x, int lp_x, int splits_x, const mfma::Params &w,
                        int splits_w, bool deep, hipStream_t s, bool w_leads, const BiasSum *bias);
// The same for 64 x 64 tiles with 4 wavefronts on both products (pooled fused epilogue only).
hipError_t mfma_pair_64x64(const mfma::Params &x, GemmOut out_x, int lp_x, int splits_x, const mfma::Params &w, int splits_w,
                           bool deep, hipStream_t s, bool w_leads, const BiasSum *bias);

}  // namespace lbp
