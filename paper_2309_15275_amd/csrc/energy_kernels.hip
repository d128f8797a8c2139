// Energy of every WHT basis of a tensor (Section 3.2, low-heuristic-error selection; the spectrum
// of Section 4.5): E[j] = sum over patches and channels of (coefficient j)^2.
//
// Patches of 2, 4 and 8: one pass over the tensor.  The coefficients of all p^2 bases are formed, squared and
// added up without leaving the registers, so the pass is bound by reading the tensor once.  (Writing the
// coefficients and reading them back moved three times the bytes: 62 us a call at 16384 tokens x 3072 bf16
// channels, 100 MB.)
//   bf16   energy_mfma_kernel: the +-1 matrix times the patch on the matrix cores
//   fp32   energy_reg_kernel: a butterfly per lane
// Patch 16 has 256 bases, more sums than a lane can hold: its coefficients are produced by the projection
// kernels (row q*256 + j of the coefficient matrix is basis j of patch q) and squared by energy_partial_kernel.
//
// Every workgroup leaves p^2 partial sums.  In the one-pass kernels the last workgroup of every 32 to arrive adds those of its 32,
// and the last of these the rest, on counters that belong to the workspace (energy_add_kernel does it for a workspace without
// counters, energy_final_kernel for patch 16).  Sums are formed in a fixed order (fp32 over at
// most 128 squares, 8 of fp32 tensors, a lane's share of a row for patch 16, then fp64), so the result is repeatable run to run.
#include "device_utils.h"
#include "kernels.h"
#include "launch.h"
#include "wht_device.h"
#include "wht_mfma_device.h"

#include <type_traits>

namespace lbp {
namespace {

constexpr int kEnergyThreads = 256;

// ---- the end of a one-pass kernel ------------------------------------------------------------------------------
//
// A launch of its own for the final sums took 4.6 us and the gap in front of it.  Calls with it / without: 1 image 16 x 16 x 768 bf16
// 6.7 / 4.9 us, 16 images 7.0 / 6.6, 64 images x 3072 (1024 workgroups) 23.6 / 22.5, fp32 1 image x 64 8.4 / 6.5.  Groups of 64
// wait for each other longer (a counter takes an arrival in about 35 ns: 4 images 7.0 us, 6.2 with groups of 32).
constexpr int kArriveGroup = 32;      // workgroups that share a counter; kEnergyMaxGroups / kArriveGroup of those share the last one
constexpr int kSetCounters = (kEnergyMaxGroups / kArriveGroup + 1) * kCounterPitch;
// One set for each workspace that has one (CounterSets), because launches that overlap in time would count each other's arrivals:
// zero between launches.
__device__ unsigned energy_counters[CounterSets::kSets * kSetCounters];

struct EnergyEnd {
    double *energy;
    int add;                     // to what it holds
    int set;                     // of energy_counters; -1: none, energy_add_kernel follows
    unsigned char nat[64];       // natural index of basis k
};

// True for the last of `n` workgroups to get here, which sees what the others have stored with device scope.
__device__ __forceinline__ bool arrive_last(unsigned *counter, unsigned n, unsigned *shared)
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);          // every lane's stores have arrived before the workgroup counts itself in
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned before = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (before == n - 1) __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *shared = before;
    }
    __syncthreads();
    const bool last = *shared == n - 1;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    return last;
}

// Device scope: sums go from one XCD's L2 to another's.
__device__ __forceinline__ void put_sum(double *p, double v)
{
    __hip_atomic_store(reinterpret_cast<unsigned long long *>(p), (unsigned long long)__double_as_longlong(v), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}

// Sum j = thread % P2 of `count` rows of sums, `pitch` values apart; the result in the first P2 of 256 threads, additions in a fixed
// order.  red: 256 values of LDS.
template <int P2>
__device__ __forceinline__ double add_rows(const double *first, int count, int pitch, double *red)
{
    constexpr int WAYS = 256 / P2;
    const int tid = threadIdx.x, j = tid % P2, way = tid / P2;
    double t = 0.0;
    for (int m = way; m < count; m += 8 * WAYS) {
        unsigned long long v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            v[u] = m + u * WAYS < count ? __hip_atomic_load(reinterpret_cast<const unsigned long long *>(first) + (size_t)(m + u * WAYS) * pitch + j,
                                                            __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0ull;
#pragma unroll
        for (int u = 0; u < 8; ++u) t += __longlong_as_double((long long)v[u]);
    }
    __syncthreads();
    red[tid] = t;
    __syncthreads();
    t = 0.0;
    for (int w = 0; w < WAYS; ++w) t += red[w * P2 + j];
    return t;
}

// The result, from the first P2 threads.
template <int P2>
__device__ __forceinline__ void store_energy(double s, const EnergyEnd &end, double *red)
{
    const int tid = threadIdx.x;
    __syncthreads();
    if (tid < P2) red[tid] = s;
    __syncthreads();
    if (tid < P2) {
        s = red[end.nat[tid]];
        end.energy[tid] = end.add ? end.energy[tid] + s : s;
    }
}

// Adds up the workgroups' sums: thread j < P2 of 256 brings sum j in natural order.  partial: P2 values a workgroup.  red: 257 values of
// LDS that nobody uses any more (and no LDS besides: four workgroups fill a unit's to the byte).  The order of all additions is fixed.
template <int P2>
__device__ __forceinline__ void finish_energy(double s, double *partial, const EnergyEnd &end, double *red)
{
    unsigned &before = *reinterpret_cast<unsigned *>(red + 256);
    unsigned *const counters = energy_counters + (size_t)max(end.set, 0) * kSetCounters;
    const int tid = threadIdx.x;
    const int groups = ((int)gridDim.x + kArriveGroup - 1) / kArriveGroup, mine = (int)blockIdx.x / kArriveGroup;
    const int members = min(kArriveGroup, (int)gridDim.x - mine * kArriveGroup);
    double *const own = partial + (size_t)mine * kArriveGroup * P2;
    if (__builtin_expect(end.set < 0 && gridDim.x > 1, 0)) {
        if (tid < P2) put_sum(partial + (size_t)blockIdx.x * P2 + tid, s);
        return;
    }
    if (members > 1) {
        if (tid < P2) put_sum(partial + (size_t)blockIdx.x * P2 + tid, s);
        if (!arrive_last(counters + (1 + mine) * kCounterPitch, members, &before)) return;
        s = add_rows<P2>(own, members, P2, red);
    }
    if (groups > 1) {            // (the first member's place is free: all of them have been read)
        if (tid < P2) put_sum(own + tid, s);
        if (!arrive_last(counters, groups, &before)) return;
        s = add_rows<P2>(partial, groups, kArriveGroup * P2, red);
    }
    store_energy<P2>(s, end, red);
}

// The same sums in the same order without counters: every workgroup adds `rows` (the last one what is left) of `count` rows of sums,
// `pitch` values apart, into the first of its rows; a single workgroup has the result.
template <int P2>
__global__ __launch_bounds__(256) void energy_add_kernel(double *partial, int count, int rows, int pitch, EnergyEnd end)
{
    __shared__ double red[256];
    double *const own = partial + (size_t)blockIdx.x * rows * pitch;
    const int members = min(rows, count - (int)blockIdx.x * rows), tid = threadIdx.x;
    if (members == 1 && gridDim.x > 1) return;
    const double s = add_rows<P2>(own, members, pitch, red);
    if (gridDim.x > 1) {
        if (tid < P2) put_sum(own + tid, s);
        return;
    }
    store_energy<P2>(s, end, red);
}

// ---- bf16, patches of 2, 4 and 8 ---------------------------------------------------------------------------
//
// One item is 64 tokens x 128 channels = 16 KB: one 8 x 8 patch, or 4 / 16 consecutive smaller ones.  Two items
// are on their way from HBM per workgroup (stage registers) while a third is multiplied out of one of two LDS
// buffers, one barrier per item; four workgroups fit a compute unit (40 KB of LDS each), 128 KB in flight.
//   8 x 8   token t = 16 ks + 8 kg + e, basis j = 32 mt + column: parity(j & t) splits by the bits of j, so the
//           product over the lower half of the tokens and that over the upper half give both column tiles as
//           their sum and their difference, and one 16-deep sign operand and its copy for odd ks serve all.
//   4 x 4   one k-step holds one patch, 2 x 2: four patches; the columns of other patches have zero signs.
//
// LINES: rows of tokens are whole 128-byte lines, which are read once and need not stay in the caches.  In others two items share a
// line, and it is to be there for the second: 64 images 16 x 16 x 3080 28.3 -> 25.5 us, 62 images 20 x 20 x 3064 40.0 -> 35.8 (whole
// lines without the hint: 64 images 16 x 16 x 3072 22.5 -> 24.1).
template <int LP, bool LINES>
__global__ __launch_bounds__(256, 4) void energy_mfma_kernel(const unsigned short *__restrict__ in, int C, int chunks,
                                                             unsigned items, GridGeom g, unsigned Q, int items_per_wg,
                                                             double *partial, EnergyEnd last)
{
    constexpr int P = 1 << LP, P2 = P * P, PATCHES = 64 / P2;
    constexpr int BUF = 64 * S_IN;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int li = lane & 31, kg = lane >> 5;

    bf16x8_t sgn_even, sgn_odd;
    {
        u16x8_t e0, e1;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const unsigned t = (unsigned)(kg * 8 + e);
            if (LP == 3) {
                e0[e] = (__popc((unsigned)li & t) & 1) ? kMinusOne : kPlusOne;
                e1[e] = (__popc((unsigned)li & (t + 16)) & 1) ? kMinusOne : kPlusOne;
            } else {
                const bool mine = li < 16 && (t / P2) == (unsigned)li / P2;
                e0[e] = !mine ? (unsigned short)0 : (__popc((unsigned)li & t & (P2 - 1)) & 1) ? kMinusOne : kPlusOne;
                e1[e] = e0[e];
            }
        }
        sgn_even = __builtin_bit_cast(bf16x8_t, e0);
        sgn_odd = __builtin_bit_cast(bf16x8_t, e1);
    }

    const int cc8 = (tid & 15) * 8;
    const int tk0 = tid >> 4;
    // lane's token of load j is row tk0 + 16 j of the item
    auto fetch = [&](unsigned group, int chunk, u32x4_t (&st)[4]) {
        const int c = chunk * CB + cc8;
        long n;
        int a0, b0;
        if (LP == 3) {
            g.origin((long)group, n, a0, b0);
            const unsigned short *base = in + g.token(n, a0, b0) * C + c;
            const int hv = c < C ? g.Ht - a0 : 0, wv = g.Wt - b0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int h = (tk0 >> 3) + 2 * j, w = tk0 & 7;
                u32x4_t v = {0u, 0u, 0u, 0u};           // zero padding past the grid or the channels
                if (h < hv && w < wv)
                    v = load_tokens<LINES>(base + ((size_t)h * g.Wt + w) * C);
                st[j] = v;
            }
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int tk = tk0 + 16 * j, t = tk & (P2 - 1), h = t >> LP, w = t & (P - 1);
                const unsigned q = group * PATCHES + (unsigned)(tk / P2);
                u32x4_t v = {0u, 0u, 0u, 0u};
                if (q < Q && c < C) {
                    g.origin((long)q, n, a0, b0);
                    if (a0 + h < g.Ht && b0 + w < g.Wt)
                        v = load_tokens<LINES>(in + g.token(n, a0 + h, b0 + w) * C + c);
                }
                st[j] = v;
            }
        }
    };

    float s0 = 0.f, s1 = 0.f;
    double t0 = 0.0, t1 = 0.0;
    auto squares = [](const f32x16_t &a) {
        float q0 = 0.f, q1 = 0.f;
#pragma unroll
        for (int e = 0; e < 16; e += 2) {
            q0 = fmaf(a[e], a[e], q0);
            q1 = fmaf(a[e + 1], a[e + 1], q1);
        }
        return q0 + q1;
    };
    auto multiply = [&](const unsigned char *buf) {
        f32x16_t lo, hi;
#pragma unroll
        for (int e = 0; e < 16; ++e) lo[e] = hi[e] = 0.f;
        if (LP == 3) {
            lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_b_frag(buf, 0, wave, lane), sgn_even, lo, 0, 0, 0);
            lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_b_frag(buf, 1, wave, lane), sgn_odd, lo, 0, 0, 0);
            hi = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_b_frag(buf, 2, wave, lane), sgn_even, hi, 0, 0, 0);
            hi = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_b_frag(buf, 3, wave, lane), sgn_odd, hi, 0, 0, 0);
            s0 += squares(lo + hi);
            s1 += squares(lo - hi);
        } else {
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
                s0 += squares(__builtin_amdgcn_mfma_f32_32x32x16_bf16(read_b_frag(buf, ks, wave, lane), sgn_even, lo, 0, 0, 0));
        }
    };

    unsigned item = blockIdx.x * (unsigned)items_per_wg;
    const unsigned end = min(items, item + (unsigned)items_per_wg);
    unsigned group = item / (unsigned)chunks;
    int chunk = (int)(item - group * (unsigned)chunks);
    unsigned fetched = item;                   // next item to request
    auto fetch_next = [&](u32x4_t (&st)[4]) {
        if (fetched >= end) return;
        fetch(group, chunk, st);
        ++fetched;
        if (++chunk == chunks) {
            chunk = 0;
            ++group;
        }
    };
    u32x4_t st[2][4];
    fetch_next(st[0]);
    fetch_next(st[1]);
    auto step = [&](u32x4_t (&cur)[4], unsigned char *buf) {
#pragma unroll
        for (int j = 0; j < 4; ++j) *reinterpret_cast<u32x4_t *>(buf + (tk0 + 16 * j) * S_IN + (tid & 15) * 16) = cur[j];
        fetch_next(cur);
        __syncthreads();     // (the buffer written next was last read before the barrier of the item in between)
        multiply(buf);
    };
    for (int i = 0; item < end; ++item, ++i) {
        if (i & 1) step(st[1], smem + BUF);
        else step(st[0], smem);
        if ((i & 7) == 7) {      // 128 squares per sum at most before it goes to double precision
            t0 += (double)s0;
            t1 += (double)s1;
            s0 = s1 = 0.f;
        }
    }
    t0 += (double)s0;
    t1 += (double)s1;
    // lanes li and li + 32 hold the same bases; then the four wavefronts, then (small patches) the patches
    t0 += __shfl_xor(t0, 32);
    t1 += __shfl_xor(t1, 32);
    __syncthreads();
    double *red = reinterpret_cast<double *>(smem);
    if (kg == 0) {
        red[wave * 64 + li] = t0;
        red[wave * 64 + 32 + li] = t1;
    }
    __syncthreads();
    double s = 0.0;
    if (tid < P2) {
#pragma unroll
        for (int w = 0; w < 4; ++w)
#pragma unroll
            for (int q = 0; q < (LP == 3 ? 1 : 16 / P2); ++q) s += red[w * 64 + q * P2 + tid];
    }
    finish_energy<P2>(s, partial, last, red + 256);
}

// ---- fp32, patches of 2, 4 and 8 ---------------------------------------------------------------------------
//
// One lane transforms one (patch, channel) at a time and keeps p^2 sums of squares.  At the end the 64 lanes
// of a wavefront add their sums by halving: every exchange with lane ^ h hands over half of the sums a lane
// still holds, so that 64 sums over 64 lanes take 63 exchanges and not 64 x 6.  A sum holds 8 squares at most before it
// goes to double precision that way.
template <int NC>
__device__ __forceinline__ double sum_by_halving(const float (&acc)[NC], int lane)
{
    double d[NC > 1 ? NC / 2 : 1];
    const bool up = (lane & 32) != 0;
#pragma unroll
    for (int i = 0; i < NC / 2; ++i) {
        const float keep = up ? acc[i + NC / 2] : acc[i], give = up ? acc[i] : acc[i + NC / 2];
        d[i] = (double)keep + (double)__shfl_xor(give, 32);
    }
    int mask = 16;
#pragma unroll
    for (int h = NC / 4; h >= 1; h >>= 1) {
        const bool u = (lane & mask) != 0;
#pragma unroll
        for (int i = 0; i < h; ++i) {
            const double keep = u ? d[i + h] : d[i], give = u ? d[i] : d[i + h];
            d[i] = keep + __shfl_xor(give, mask);
        }
        mask >>= 1;
    }
    double s = d[0];
    for (; mask >= 1; mask >>= 1) s += __shfl_xor(s, mask);
    return s;
}

// SHORT: up to 8 rounds, which need no outer loop (64 images 56 x 56 x 96 in 4 x 4 patches, 3 rounds: 18.0 us, 18.4 with it).
template <int LP, bool SHORT>
__global__ __launch_bounds__(256) void energy_reg_kernel(const float *__restrict__ in, int C, unsigned long items, GridGeom g,
                                                         int rounds, double *partial, EnergyEnd last)
{
    constexpr int P = 1 << LP, NC = P * P, KEEP = 64 / NC;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    float acc[NC];
    double s = 0.0;                          // basis lane / KEEP
    unsigned long item = (unsigned long)blockIdx.x * rounds * 256 + tid;
    for (int done = 0; done < rounds; done += 8) {       // (the same for every lane)
#pragma unroll
        for (int j = 0; j < NC; ++j) acc[j] = 0.f;
        const int until = SHORT ? rounds : min(rounds, done + 8);
        for (int it = done; it < until && item < items; ++it, item += 256) {
            const unsigned q = items <= 0xffffffffUL ? (unsigned)item / (unsigned)C : (unsigned)(item / C);
            const int c = (int)(item - (unsigned long)q * C);
            long img;
            int a0, b0;
            g.origin((long)q, img, a0, b0);
            const float *src = in + g.token(img, a0, b0) * C + c;
            const int hv = g.Ht - a0, wv = g.Wt - b0;
            float v[NC];
            if (hv >= P && wv >= P) {       // the whole patch is inside the grid
#pragma unroll
                for (int j = 0; j < NC; ++j) v[j] = __builtin_nontemporal_load(src + ((size_t)(j >> LP) * g.Wt + (j & (P - 1))) * C);
            } else {
#pragma unroll
                for (int j = 0; j < NC; ++j) {
                    v[j] = 0.f;
                    if ((j >> LP) < hv && (j & (P - 1)) < wv) v[j] = __builtin_nontemporal_load(src + ((size_t)(j >> LP) * g.Wt + (j & (P - 1))) * C);
                }
            }
            fwht_inplace<NC>(v);
#pragma unroll
            for (int j = 0; j < NC; ++j) acc[j] = fmaf(v[j], v[j], acc[j]);
        }
        s += sum_by_halving<NC>(acc, lane);
        if (SHORT) break;
    }
    __shared__ double red[256], all[257];
    if (lane % KEEP == 0) red[wave * NC + lane / KEEP] = s;
    __syncthreads();
    s = tid < NC ? (red[tid] + red[NC + tid]) + (red[2 * NC + tid] + red[3 * NC + tid]) : 0.0;
    finish_energy<NC>(s, partial, last, all);
}

// ---- patch 16: squares of coefficients that a projection kernel wrote ---------------------------------------

// grid (p^2, NB): workgroup (j, b) covers basis j of patches [b*per, (b+1)*per)
template <bool BF16>
__global__ __launch_bounds__(kEnergyThreads) void energy_partial_kernel(const void *__restrict__ coef, long Q,
                                                                       int pp, int C, long per,
                                                                       double *__restrict__ partial)
{
    __shared__ double red[kEnergyThreads];
    const int j = blockIdx.x, b = blockIdx.y;
    const long q0 = (long)b * per, q1 = min(Q, q0 + per);
    const int vecs = BF16 ? C / 8 : C / 4;      // 16-byte vectors per row
    double total = 0.0;
    for (long q = q0; q < q1; ++q) {
        const uint4 *row = reinterpret_cast<const uint4 *>(coef) + ((size_t)q * pp + j) * vecs;
        float s = 0.f;
        for (int v = threadIdx.x; v < vecs; v += kEnergyThreads) {
            uint4 u = row[v];
            if (BF16) {
                float f[8] = {bf16_lo_to_f32(u.x), bf16_hi_to_f32(u.x), bf16_lo_to_f32(u.y), bf16_hi_to_f32(u.y),
                              bf16_lo_to_f32(u.z), bf16_hi_to_f32(u.z), bf16_lo_to_f32(u.w), bf16_hi_to_f32(u.w)};
#pragma unroll
                for (int e = 0; e < 8; ++e) s = fmaf(f[e], f[e], s);
            } else {
                float f[4] = {__uint_as_float(u.x), __uint_as_float(u.y), __uint_as_float(u.z), __uint_as_float(u.w)};
#pragma unroll
                for (int e = 0; e < 4; ++e) s = fmaf(f[e], f[e], s);
            }
        }
        total += (double)s;
    }
    red[threadIdx.x] = total;
    __syncthreads();
    for (int h = kEnergyThreads / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[(size_t)j * gridDim.y + b] = red[0];
}

// energy[k] (+)= sum_b partial[row.v[k]][b], one workgroup per basis, fixed order
__global__ __launch_bounds__(256) void energy_final_kernel(const double *__restrict__ partial, int nb, NatTable row, int add,
                                                           double *energy)
{
    __shared__ double red[4];
    const double *src = partial + (size_t)row.v[blockIdx.x] * nb;
    double s = 0.0;
    for (int b = threadIdx.x; b < nb; b += 256) s += src[b];
#pragma unroll
    for (int h = 32; h >= 1; h >>= 1) s += __shfl_xor(s, h);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        s = (red[0] + red[1]) + (red[2] + red[3]);
        energy[blockIdx.x] = add ? energy[blockIdx.x] + s : s;
    }
}

int energy_chunks(long Q)
{
    long nb = Q < 64 ? Q : 64;
    return (int)(nb < 1 ? 1 : nb);
}

size_t coef_bytes(long Q, int pp, int C, int dtype) { return ((size_t)Q * pp * C * dtype_size(dtype) + 255) / 256 * 256; }

// The split of a one-pass kernel: workgroups (each leaves p^2 partial sums) and items of a workgroup (bf16) or of a lane (fp32).
struct EnergySplit {
    unsigned long items;
    int per, groups;
};

EnergySplit energy_split(long Q, int C, int dtype, int lp)
{
    EnergySplit s;
    if (dtype == LBP_BF16) {
        s.items = (unsigned long)(((Q << (2 * lp)) + 63) / 64) * (unsigned long)((C + CB - 1) / CB);
        // four workgroups per compute unit of an MI355X are resident; a longer run of items per workgroup rather than more of them
        s.per = (int)((s.items + 1023) / 1024);
        s.groups = (int)((s.items + s.per - 1) / s.per);
    } else {
        s.items = (unsigned long)Q * C;
        const unsigned long blocks = (s.items + 255) / 256;
        s.per = (int)((blocks + kEnergyMaxGroups - 1) / kEnergyMaxGroups);
        s.groups = (int)((blocks + s.per - 1) / s.per);
    }
    return s;
}

template <int LP>
hipError_t launch_one_pass(const void *in, long Q, int C, int dtype, const GridGeom &g, double *partial, const EnergyEnd &last,
                           hipStream_t stream)
{
    const EnergySplit s = energy_split(Q, C, dtype, LP);
    const dim3 grid((unsigned)s.groups);
    if (s.groups > kEnergyMaxGroups || last.set >= CounterSets::kSets) return hipErrorInvalidValue;
    hipError_t e;
    if (dtype == LBP_BF16) {
        static_assert(2 * 64 * S_IN >= (2 * 256 + 1) * (int)sizeof(double), "the final sums fit the staging buffers");
        auto launch = [&](auto lines) {
            return LBP_LAUNCH_KERNEL((energy_mfma_kernel<LP, decltype(lines)::value>), grid, 256, 2 * 64 * S_IN, stream,
                                     (const unsigned short *)in, C, (C + CB - 1) / CB, (unsigned)s.items, g, (unsigned)Q, s.per, partial, last);
        };
        e = C % 64 == 0 ? launch(std::true_type{}) : launch(std::false_type{});
    } else if (s.per <= 8) {
        e = LBP_LAUNCH_KERNEL((energy_reg_kernel<LP, true>), grid, 256, 0, stream, (const float *)in, C, s.items, g, s.per, partial, last);
    } else {
        e = LBP_LAUNCH_KERNEL((energy_reg_kernel<LP, false>), grid, 256, 0, stream, (const float *)in, C, s.items, g, s.per, partial, last);
    }
    if (e != hipSuccess || last.set >= 0 || s.groups < 2) return e;
    constexpr int P2 = 1 << (2 * LP);
    const int groups = (s.groups + kArriveGroup - 1) / kArriveGroup;
    e = LBP_LAUNCH_KERNEL(energy_add_kernel<P2>, dim3((unsigned)groups), 256, 0, stream, partial, s.groups, kArriveGroup, P2, last);
    if (e != hipSuccess || groups < 2) return e;
    return LBP_LAUNCH_KERNEL(energy_add_kernel<P2>, dim3(1), 256, 0, stream, partial, groups, groups, kArriveGroup * P2, last);
}

}  // namespace

size_t energy_workspace_bytes(long Q, int C, int dtype, int patch)
{
    const int pp = patch * patch;
    if (patch <= 8) return (size_t)pp * energy_split(Q, C, dtype, patch == 8 ? 3 : patch == 4 ? 2 : 1).groups * sizeof(double);
    return coef_bytes(Q, pp, C, dtype) + (size_t)pp * energy_chunks(Q) * sizeof(double);
}

hipError_t launch_energy(const void *in, int N, int H, int W, int C, int dtype, const BasisPlan &all, WhtPath path, int extra,
                         char *workspace, int counter_set, double *energy, bool add, hipStream_t stream)
{
    const int patch = all.patch, pp = patch * patch;
    const long Q = patch_count(N, H, W, patch);
    const GridGeom g = make_geom(H, W, patch, extra);
    double *partial = reinterpret_cast<double *>(workspace);
    if (patch <= 8) {
        EnergyEnd last{energy, add ? 1 : 0, counter_set, {}};
        for (int k = 0; k < pp; ++k) last.nat[k] = all.nat[k];
        if (patch == 8) return launch_one_pass<3>(in, Q, C, dtype, g, partial, last, stream);
        if (patch == 4) return launch_one_pass<2>(in, Q, C, dtype, g, partial, last, stream);
        return launch_one_pass<1>(in, Q, C, dtype, g, partial, last, stream);
    }
    NatTable row;
    int nb = 0;
    hipError_t e;
    {
        e = launch_project(in, workspace, N, H, W, C, dtype, all, path, stream, extra, 0.0f);
        if (e != hipSuccess) return e;
        partial = reinterpret_cast<double *>(workspace + coef_bytes(Q, pp, C, dtype));
        nb = energy_chunks(Q);
        const long per = (Q + nb - 1) / nb;
        dim3 grid((unsigned)pp, (unsigned)nb);
        if (dtype == LBP_BF16)
            hipLaunchKernelGGL(energy_partial_kernel<true>, grid, dim3(kEnergyThreads), 0, stream, workspace, Q, pp, C, per, partial);
        else
            hipLaunchKernelGGL(energy_partial_kernel<false>, grid, dim3(kEnergyThreads), 0, stream, workspace, Q, pp, C, per, partial);
        e = hipGetLastError();
        for (int k = 0; k < kMaxBases; ++k) row.v[k] = (uint8_t)k;
    }
    if (e != hipSuccess) return e;
    return LBP_LAUNCH_KERNEL(energy_final_kernel, dim3((unsigned)pp), 256, 0, stream, partial, nb, row, add ? 1 : 0, energy);
}

}  // namespace lbp
