// fp32 matrix products of the backward pass on the fp32 matrix cores (v_mfma_f32_32x32x2_f32: fp32 operands,
// fp32 accumulation, 256 clocks per 64 x 64 x 4 block of a compute unit, 157 TFLOP/s on the chip).
//
// One launch runs the input-gradient product (A = g^y stored [M][K], rows are (patch, basis) pairs or tokens), the
// weight-gradient product (A = g^y stored [K][M]), or both: they only share the read-only g^y.
//   * A workgroup (4 wavefronts, 2 x 2) owns a BM x 64 tile, BM = 64, or 128 for the input gradient where whole
//     patches of r rows fill 128 better than 64.  A lone 64 x 64 x 32 step is 0.43 us of matrix-core time and moves
//     16 KB; three workgroups (165 registers, 37 KB of LDS each) share a compute unit and cover each other's waits.
//   * Global -> registers (PF steps ahead) -> LDS (two stages, one barrier per step).  Reduction-fast operands are
//     kept [row][k] and read 16 bytes a lane: lane half kg takes k = 8 s + 4 kg + j as its value of instruction j.
//     Reduction-slow operands are kept [k][row] and read 4 bytes a lane with the same k per instruction.
//   * A product with few tiles is cut along its reduction; the slices of a tile leave their partial sums in device
//     memory and the last one to arrive adds them in slice order (no workgroup waits, results do not depend on
//     who came last) and runs the epilogue, so no reduction kernel follows.
//   * The input gradient's epilogue applies p^-1(.) of Eq. 7 to the tile's patches and stores tokens.
// Against the FMA kernel this replaced (gemm_kernels.hip keeps it as the cross-check): 640 rows, 768 <-> 3072
// channels, r = 10: 119 + 163 us for the two products and 12 us for the reverse projection.
#include "device_utils.h"
#include "kernels.h"
#include "launch.h"
#include "wht_device.h"

namespace lbp {
namespace {

typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int BN = 64, BK = 32;
constexpr int S_KFAST = BK + 4;      // LDS row pitch of a [row][k] tile in floats: 16-byte reads of 8 rows cover all banks
constexpr int S_CT = BN + 4;         // pitch of the accumulators in LDS (epilogue)

struct F32Product {
    const float *A, *B;
    float *C;
    int M, N, K, lda, ldb;
    int k_per_split;     // multiple of BK
    int splits;
    int tiles_m, tiles_n;
    int bm_step;         // rows one tile advances by
    float scale;
    float *parts;        // [tile][slice][BM * 64]
    unsigned *counters;  // one per tile, zero between launches
};

struct F32Tokens {       // the input gradient's epilogue (r = 0: plain store)
    GridGeom geom;
    PooledSel sel;
    int r, lp, mh, mw;
    long Q;
    int extra_rows, extra;
    unsigned char nat[66];   // natural index of every selected basis (8 x 8 patches; read in pairs)
};

struct F32Params {
    F32Product x, w;
    F32Tokens tok;
    unsigned blocks_first, blocks_x;     // workgroups of the product that is dispatched first; of x
    int w_first;
};

// Tokens of the tile's patches from the coefficients in ct[row][S_CT], patches of 2 and 4: one (patch, channel) per
// lane, butterfly of at most 16 values in registers.
template <int LP, int MH, int MW>
__device__ __forceinline__ void store_tokens(const float *ct, const F32Tokens &t, float *out, int N, int bm_step, int m0,
                                             int n0, int tid)
{
    constexpr int P = 1 << LP, PWd = P >> MW, NC = (P >> MH) * PWd;
    constexpr float scale = 1.0f / (float)(P * P);
    const int patches = bm_step / t.r;
    for (int it = tid; it < patches * BN; it += 256) {
        const int pt = it >> 6, c = it & 63;
        const long q = (long)(m0 / t.r) + pt;
        if (q >= t.Q || n0 + c >= N) continue;
        const float *src = ct + (size_t)(pt * t.r) * S_CT + c;
        float v[NC];
#pragma unroll
        for (int j = 0; j < NC; ++j) v[j] = (t.sel.mask >> j) & 1ull ? src[t.sel.pos[j] * S_CT] : 0.f;
        fwht_inplace<NC>(v);
        long img;
        int a0, b0;
        t.geom.origin(q, img, a0, b0);
        float *dst = out + t.geom.token(img, a0, b0) * N + n0 + c;
        const int hv = t.geom.Ht - a0, wv = t.geom.Wt - b0;
#pragma unroll
        for (int h = 0; h < P; ++h)
#pragma unroll
            for (int w = 0; w < P; ++w)
                if (h < hv && w < wv)
                    __builtin_nontemporal_store(v[(h >> MH) * PWd + (w >> MW)] * scale, dst + ((size_t)h * t.geom.Wt + w) * N);
    }
}

// The same for 8 x 8 patches: tokens[64][64] = S[64][r] coefficients[r][64] on the matrix cores, S the +-1 matrix; each
// wavefront a quarter of every patch.  r / 2 instructions per patch against a 64-value butterfly per lane, whose
// register arrays would leave the product half its wavefronts.
__device__ __forceinline__ void store_tokens_8x8(const float *ct, const F32Tokens &t, float *out, int N, int bm_step, int m0,
                                                 int n0, int wm, int wn, int li, int kg)
{
    const int r = t.r, patches = bm_step / r, pairs = (r + 1) >> 1;
    const unsigned tk = (unsigned)(wm * 32 + li);
    unsigned neg = 0;                        // bit s: sign of this lane's token under basis 2 s + kg
    for (int s = 0; s < pairs; ++s) {
        const unsigned nat = kg ? t.nat[2 * s + 1] : t.nat[2 * s];
        neg |= (unsigned)(__popc(nat & tk) & 1) << s;
    }
    const int col = n0 + wn * 32 + li;
    for (int pt = 0; pt < patches; ++pt) {
        const long q = (long)(m0 / r) + pt;
        if (q >= t.Q) break;
        const float *src = ct + (pt * r + kg) * S_CT + wn * 32 + li;
        f32x16_t o;
#pragma unroll
        for (int e = 0; e < 16; ++e) o[e] = 0.f;
        int s = 0;
        for (; s + 4 <= (r >> 1); s += 4) {
            float c[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) c[u] = src[2 * (s + u) * S_CT];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                o = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(0x3f800000u | ((neg >> (s + u)) << 31)), c[u], o, 0, 0, 0);
        }
        for (; s < pairs; ++s) {             // (an odd r: the other half of the last pair must not be read as anything but zero)
            const float c = 2 * s + kg < r ? src[2 * s * S_CT] : 0.f;
            o = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(0x3f800000u | ((neg >> s) << 31)), c, o, 0, 0, 0);
        }
        long img;
        int a0, b0;
        t.geom.origin(q, img, a0, b0);
        // element e: token row 4 wm + e / 4, token column 4 kg + e % 4
        const int hv = col < N ? t.geom.Ht - a0 - wm * 4 : 0, wv = t.geom.Wt - b0 - kg * 4;
        float *dst = out + t.geom.token(img, a0 + wm * 4, b0 + kg * 4) * N + col;
#pragma unroll
        for (int e = 0; e < 16; ++e)
            if ((e >> 2) < hv && (e & 3) < wv)
                __builtin_nontemporal_store(o[e] * (1.0f / 64.0f), dst + ((size_t)(e >> 2) * t.geom.Wt + (e & 3)) * N);
    }
}

template <int BM, bool A_KFAST>
struct Lds {
    static constexpr int SA = A_KFAST ? S_KFAST : BM + 8, SB = BN + 8;      // k and k + 4 fall into different halves of the banks
    static constexpr int A = (A_KFAST ? BM : BK) * SA, STAGE = A + BK * SB;  // floats
    static constexpr int LOOP = 2 * STAGE * 4, EPI = BM * S_CT * 4;
    static constexpr int BYTES = LOOP > EPI ? LOOP : EPI;
};

template <int BM, bool A_KFAST, bool TOKENS>
__device__ __forceinline__ void product(const F32Product &p, const F32Tokens &tok, unsigned block, float *smem)
{
    using L = Lds<BM, A_KFAST>;
    constexpr int TM = BM / 64;                     // 32 x 32 blocks of a wavefront along M (one along N)
    constexpr int A_CH = BM * BK / 4 / 256, B_CH = BN * BK / 4 / 256;      // 16-byte pieces per lane and step
    constexpr int PF = BM == 64 ? 4 : 2;            // steps in flight
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wm = wave >> 1, wn = wave & 1;
    const int li = lane & 31, kg = lane >> 5;
    const unsigned T = (unsigned)(p.tiles_m * p.tiles_n);
    const unsigned slice = block / T;
    // workgroups go round-robin over the 8 XCDs: each XCD takes a contiguous run of tiles
    unsigned tile = block - slice * T;
    {
        const unsigned x = tile & 7, i = tile >> 3, base = T >> 3, rem = T & 7;
        tile = x * base + (x < rem ? x : rem) + i;
    }
    const int tm = (int)(tile / (unsigned)p.tiles_n), tn = (int)(tile - (unsigned)tm * p.tiles_n);
    const int m0 = tm * p.bm_step, n0 = tn * BN;
    const int kbeg = (int)slice * p.k_per_split, kend = min(p.K, kbeg + p.k_per_split);

    const float *ga[A_CH], *gb[B_CH];
    int sa[A_CH], sb[B_CH], ka[A_CH], kb[B_CH];
#pragma unroll
    for (int i = 0; i < A_CH; ++i) {
        const int c = tid + i * 256;
        if (A_KFAST) {
            const int row = c >> 3, kc = (c & 7) * 4;
            ka[i] = kc;
            sa[i] = row * L::SA + kc;
            ga[i] = p.A + (size_t)min(m0 + row, p.M - 1) * p.lda + kc;      // rows past the edge feed outputs nobody stores
        } else {
            const int k = c / (BM / 4), col = c % (BM / 4) * 4;
            ka[i] = k;
            sa[i] = k * L::SA + col;
            ga[i] = p.A + (size_t)k * p.lda + min(m0 + col, p.M - 4);
        }
    }
#pragma unroll
    for (int i = 0; i < B_CH; ++i) {
        const int c = tid + i * 256, k = c >> 4, col = (c & 15) * 4;
        kb[i] = k;
        sb[i] = L::A + k * L::SB + col;
        gb[i] = p.B + (size_t)k * p.ldb + min(n0 + col, p.N - 4);
    }
    float4 ra[PF][A_CH], rb[PF][B_CH];
    auto fetch = [&](int set, int k0) {              // a whole step
#pragma unroll
        for (int i = 0; i < A_CH; ++i) ra[set][i] = *reinterpret_cast<const float4 *>(ga[i] + (A_KFAST ? (size_t)k0 : (size_t)k0 * p.lda));
#pragma unroll
        for (int i = 0; i < B_CH; ++i) rb[set][i] = *reinterpret_cast<const float4 *>(gb[i] + (size_t)k0 * p.ldb);
    };
    auto fetch_tail = [&](int set, int k0) {         // a partial one: zeros past the end
#pragma unroll
        for (int i = 0; i < A_CH; ++i) {
            ra[set][i] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (k0 + ka[i] < kend) ra[set][i] = *reinterpret_cast<const float4 *>(ga[i] + (A_KFAST ? (size_t)k0 : (size_t)k0 * p.lda));
        }
#pragma unroll
        for (int i = 0; i < B_CH; ++i) {
            rb[set][i] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (k0 + kb[i] < kend) rb[set][i] = *reinterpret_cast<const float4 *>(gb[i] + (size_t)k0 * p.ldb);
        }
    };
    auto stage = [&](int set, float *s) {
#pragma unroll
        for (int i = 0; i < A_CH; ++i) *reinterpret_cast<float4 *>(s + sa[i]) = ra[set][i];
#pragma unroll
        for (int i = 0; i < B_CH; ++i) *reinterpret_cast<float4 *>(s + sb[i]) = rb[set][i];
    };
    f32x16_t acc[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
    auto multiply = [&](const float *s) {
#pragma unroll
        for (int g = 0; g < BK / 8; ++g) {
            float a[TM][4], b[4];
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int row = wm * (BM / 2) + i * 32 + li;
                if (A_KFAST) {
                    const float4 v = *reinterpret_cast<const float4 *>(s + row * L::SA + g * 8 + kg * 4);
                    a[i][0] = v.x; a[i][1] = v.y; a[i][2] = v.z; a[i][3] = v.w;
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) a[i][j] = s[(g * 8 + kg * 4 + j) * L::SA + row];
                }
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) b[j] = s[L::A + (g * 8 + kg * 4 + j) * L::SB + wn * 32 + li];
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int i = 0; i < TM; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][j], b[j], acc[i], 0, 0, 0);
        }
    };

    float *const bufs[2] = {smem, smem + L::STAGE};
    const int nfull = (kend - kbeg) / BK;
    if (nfull > 0) {
#pragma unroll
        for (int j = 0; j < PF; ++j)
            if (j < nfull) fetch(j, kbeg + j * BK);
        stage(0, bufs[0]);
        __syncthreads();
        // at the top of step s (j = s mod PF): stage s & 1 holds step s, sets j+1 .. j+PF-1 are on their way
        int s = 0;
        for (; s + 2 * PF - 1 < nfull; s += PF) {
#pragma unroll
            for (int j = 0; j < PF; ++j) {
                fetch(j, kbeg + (s + j + PF) * BK);
                multiply(bufs[j & 1]);
                stage((j + 1) % PF, bufs[(j + 1) & 1]);
                __syncthreads();
            }
        }
        const int rem = nfull - s;
#pragma unroll
        for (int j = 0; j < 2 * PF - 1; ++j) {
            if (j < rem) {
                if (s + j + PF < nfull) fetch(j % PF, kbeg + (s + j + PF) * BK);
                multiply(bufs[j & 1]);
                if (j + 1 < rem) stage((j + 1) % PF, bufs[(j + 1) & 1]);
                __syncthreads();
            }
        }
    }
    if (kbeg + nfull * BK < kend) {
        fetch_tail(0, kbeg + nfull * BK);
        stage(0, bufs[0]);
        __syncthreads();
        multiply(bufs[0]);
        __syncthreads();
    }

    if (p.splits > 1) {
        // The slices' sums cross from one XCD's L2 to another's: device-scope accesses, 8 bytes a lane, go to where
        // the XCDs are coherent (a fence would write back and invalidate whole caches).
        __shared__ unsigned arrived;
        constexpr int NV = TM * 8;
        unsigned long long *const parts = reinterpret_cast<unsigned long long *>(p.parts) + (size_t)tile * p.splits * (BM * BN / 2) + tid;
        unsigned long long *mine = parts + (size_t)slice * (BM * BN / 2);
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            const unsigned long long v = (unsigned long long)__float_as_uint(acc[q >> 3][2 * (q & 7)]) |
                                         ((unsigned long long)__float_as_uint(acc[q >> 3][2 * (q & 7) + 1]) << 32);
            __hip_atomic_store(mine + (size_t)q * 256, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_waitcnt(0);            // every lane's part has arrived before the workgroup counts itself in
        __syncthreads();
        if (tid == 0) arrived = __hip_atomic_fetch_add(p.counters + tile, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (arrived != (unsigned)(p.splits - 1)) return;      // the same for every lane of the workgroup
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
        constexpr int U = 2;                      // parts in flight together
        for (int z = 0; z < p.splits; z += U) {
            unsigned long long v[U][NV];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int q = 0; q < NV; ++q)
                    v[u][q] = z + u < p.splits ? __hip_atomic_load(parts + (size_t)(z + u) * (BM * BN / 2) + (size_t)q * 256,
                                                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0ull;
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int q = 0; q < NV; ++q) {
                    acc[q >> 3][2 * (q & 7)] += __uint_as_float((unsigned)v[u][q]);
                    acc[q >> 3][2 * (q & 7) + 1] += __uint_as_float((unsigned)(v[u][q] >> 32));
                }
        }
        if (tid == 0) __hip_atomic_store(p.counters + tile, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }

    // element 4 g4 + e of a block: row 8 g4 + 4 kg + e, column li
    if constexpr (TOKENS) {
        if (tok.r > 0) {
            float *ct = smem;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    ct[(wm * (BM / 2) + i * 32 + (e >> 2) * 8 + kg * 4 + (e & 3)) * S_CT + wn * 32 + li] = acc[i][e];
            __syncthreads();
            switch (tok.lp * 16 + tok.mh * 4 + tok.mw) {
#define LBP_CASE(LP, MH, MW)                                                                       \
    case LP * 16 + MH * 4 + MW:                                                                    \
        store_tokens<LP, MH, MW>(ct, tok, p.C, p.N, p.bm_step, m0, n0, tid);                       \
        break;
                LBP_CASE(1, 0, 0) LBP_CASE(1, 0, 1) LBP_CASE(1, 1, 0) LBP_CASE(1, 1, 1)
                LBP_CASE(2, 0, 0) LBP_CASE(2, 0, 1) LBP_CASE(2, 0, 2) LBP_CASE(2, 1, 0) LBP_CASE(2, 1, 1) LBP_CASE(2, 1, 2)
                LBP_CASE(2, 2, 0) LBP_CASE(2, 2, 1) LBP_CASE(2, 2, 2)
#undef LBP_CASE
                default: store_tokens_8x8(ct, tok, p.C, p.N, p.bm_step, m0, n0, wm, wn, li, kg);
            }
            if (tok.extra_rows > 0) {      // tokens outside the grid: their rows are the gradient itself, scaled
                const long first = tok.Q * tok.r;
                const int lo = (int)max(0L, min((long)p.bm_step, first - m0)), hi = (int)min((long)p.bm_step, (long)p.M - m0);
                const float inv = 1.0f / (float)(1 << (2 * tok.lp));
                for (int it = tid; it < (hi - lo) * BN; it += 256) {
                    const int lr = lo + (it >> 6), c = it & 63;
                    if (n0 + c >= p.N) continue;
                    const long j = (long)m0 + lr - first, img = j / tok.extra;
                    p.C[((size_t)img * tok.geom.img + (j - img * tok.extra)) * p.N + n0 + c] = ct[lr * S_CT + c] * inv;
                }
            }
            return;
        }
    }
    const int col = n0 + wn * 32 + li;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int row = m0 + wm * (BM / 2) + i * 32 + (e >> 2) * 8 + kg * 4 + (e & 3);
            if (row < p.M && col < p.N) p.C[(size_t)row * p.N + col] = acc[i][e] * p.scale;
        }
}

template <int BMX>
__global__ __launch_bounds__(256, 3) void gemm_f32_mfma_kernel(F32Params p)
{
    extern __shared__ __attribute__((aligned(16))) float smem_f32[];
    const bool first = blockIdx.x < p.blocks_first;
    const unsigned b = first ? blockIdx.x : blockIdx.x - p.blocks_first;
    if (first == (p.w_first != 0)) product<64, false, false>(p.w, p.tok, b, smem_f32);
    else product<BMX, true, true>(p.x, p.tok, b, smem_f32);
}

int ceil_div(long a, long b) { return (int)((a + b - 1) / b); }

// Kernel parameters of one product; false: a shape or slicing the kernel does not take.
bool fill(const GemmArgs &a, int bm, F32Product *p)
{
    if (a.dtype != LBP_F32 || a.splits < 1 || a.K < 1 || a.N < 4 || a.N % 4 || a.lda % 4 || a.ldb % 4) return false;
    // rows of a reduction-fast A are clamped one by one, the others in pieces of 4
    if (a.a_kfast ? a.M < 1 || a.K % 4 : a.M < 4 || a.M % 4) return false;
    p->A = (const float *)a.A;
    p->B = (const float *)a.B;
    p->C = (float *)a.C;
    p->M = a.M; p->N = a.N; p->K = a.K;
    p->lda = (int)a.lda; p->ldb = (int)a.ldb;
    p->k_per_split = ceil_div(ceil_div(a.K, a.splits), BK) * BK;
    p->splits = a.splits;
    p->bm_step = a.out == GemmOut::kUnproject ? f32_tile_step(a.M, a.N, a.K, a.plan->r, a.plan->patch, device_cus()) : bm;
    p->tiles_m = ceil_div(a.M, p->bm_step);
    p->tiles_n = ceil_div(a.N, BN);
    p->scale = a.scale;
    p->parts = (float *)a.join_parts;
    if (a.splits > 1) {
        if ((long)(a.splits - 1) * p->k_per_split >= a.K) return false;        // no empty slice
        if (!a.join_parts || (size_t)p->tiles_m * p->tiles_n * a.splits * bm * BN * sizeof(float) > a.join_bytes) return false;
    }
    return true;
}

}  // namespace

hipError_t launch_gemm_f32(const GemmArgs *x, const GemmArgs *w, hipStream_t stream)
{
    F32Params p{};
    int bm = 64;
    if (x) {
        if (!x->a_kfast || (x->out != GemmOut::kF32 && x->out != GemmOut::kUnproject)) return hipErrorInvalidValue;
        if (x->out == GemmOut::kUnproject) {
            if (!x->plan || x->plan->patch > 8) return hipErrorInvalidValue;
            const BasisPlan &bp = *x->plan;
            bm = f32_tile_rows(bp.r);
            if (x->extra_rows < 0 || x->extra_rows > x->M || (x->extra_rows > 0 && (x->extra < 1 || x->extra_rows % x->extra)) ||
                (x->M - x->extra_rows) % bp.r)
                return hipErrorInvalidValue;
            p.tok.geom = make_geom(x->grid_h, x->grid_w, bp.patch, x->extra);
            p.tok.sel.mask = bp.pooled_mask;
            for (int j = 0; j < 64; ++j) p.tok.sel.pos[j] = bp.pooled_pos[j];
            for (int k = 0; k < bp.r && k < 64; ++k) p.tok.nat[k] = (unsigned char)bp.nat[k];
            p.tok.r = bp.r; p.tok.lp = bp.log2p; p.tok.mh = bp.mh; p.tok.mw = bp.mw;
            p.tok.Q = (x->M - x->extra_rows) / bp.r;
            p.tok.extra_rows = x->extra_rows;
            p.tok.extra = x->extra > 0 ? x->extra : 1;
        }
        if (!fill(*x, bm, &p.x)) return hipErrorInvalidValue;
    }
    if (w && (w->a_kfast || w->out != GemmOut::kF32 || !fill(*w, 64, &p.w))) return hipErrorInvalidValue;
    if (!x && !w) return hipErrorInvalidValue;
    const long tx = x ? (long)p.x.tiles_m * p.x.tiles_n : 0, tw = w ? (long)p.w.tiles_m * p.w.tiles_n : 0;
    if ((x && p.x.splits > 1) || (w && p.w.splits > 1)) {
        if (tx + tw > kJoinMaxTiles) return hipErrorInvalidValue;
        p.x.counters = join_counter_ptr();
        if (!p.x.counters) return hipErrorInvalidSymbol;
        p.w.counters = p.x.counters + tx;
    }
    const long bx = x ? tx * p.x.splits : 0, bw = w ? tw * p.w.splits : 0;
    if (bx + bw > 0x7fffffffL) return hipErrorInvalidValue;
    // the workgroups with the longer reductions start first, the short ones fill the end of the launch
    p.w_first = w && (!x || p.w.k_per_split > p.x.k_per_split) ? 1 : 0;
    p.blocks_x = (unsigned)bx;
    p.blocks_first = (unsigned)(p.w_first ? bw : bx);
    constexpr int L64 = Lds<64, true>::BYTES > Lds<64, false>::BYTES ? Lds<64, true>::BYTES : Lds<64, false>::BYTES;
    constexpr int L128 = Lds<128, true>::BYTES > L64 ? Lds<128, true>::BYTES : L64;
    if (bm == 64) return LBP_LAUNCH_KERNEL(gemm_f32_mfma_kernel<64>, dim3((unsigned)(bx + bw)), 256, L64, stream, p);
    return LBP_LAUNCH_KERNEL(gemm_f32_mfma_kernel<128>, dim3((unsigned)(bx + bw)), 256, L128, stream, p);
}

}  // namespace lbp
