// Pieces the matrix-core WHT kernels share: operand types, the LDS layout of a [k][channel] tile read with the
// transposing LDS read, and the sign operands.
#pragma once
#include "device_utils.h"

namespace lbp {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef short i16x4_t __attribute__((ext_vector_type(4)));
typedef unsigned short u16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));   // 16 bytes, usable with the non-temporal builtins

#define LBP_LDS_PTR(T, p) ((__attribute__((address_space(3))) T *)(p))

constexpr int CB = 128;                 // channels per workgroup item
constexpr int S_IN = CB * 2 + 64;       // LDS row pitch of a [k][channel] bf16 tile read with tr16_b64
constexpr int S_OUT = CB * 2 + 16;      // LDS row pitch of the staged result rows
constexpr unsigned short kPlusOne = 0x3F80, kMinusOne = 0xBF80;

// 16 bytes of a token.  LINES: tokens are whole 128-byte lines, which are read once and need not stay in the caches.
template <bool LINES>
__device__ __forceinline__ u32x4_t load_tokens(const unsigned short *p)
{
    const u32x4_t *v = reinterpret_cast<const u32x4_t *>(p);
    if constexpr (LINES) return __builtin_nontemporal_load(v);
    else return *v;
}

// 8 consecutive reduction entries of one row of the sign matrix, as a matrix-core operand.
// forward:  row = basis (natural index `fixed`), entries = tokens t0..t0+7
// reverse:  row = token `fixed`, entries = bases k0..k0+7 (natural indices from the LDS table)
__device__ __forceinline__ bf16x8_t signs_over_tokens(unsigned nat, int t0, int p2, bool row_ok)
{
    u16x8_t v;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        int t = t0 + e;
        unsigned short s = (__popc(nat & (unsigned)t) & 1) ? kMinusOne : kPlusOne;
        v[e] = (row_ok && t < p2) ? s : (unsigned short)0;
    }
    return __builtin_bit_cast(bf16x8_t, v);
}

__device__ __forceinline__ bf16x8_t signs_over_bases(const unsigned char *lds_nat, int k0, int r, unsigned t,
                                                     bool row_ok)
{
    u16x8_t v;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        int k = k0 + e;
        unsigned nat = lds_nat[k < r ? k : 0];
        unsigned short s = (__popc(nat & t) & 1) ? kMinusOne : kPlusOne;
        v[e] = (row_ok && k < r) ? s : (unsigned short)0;
    }
    return __builtin_bit_cast(bf16x8_t, v);
}

// B operand (reduction index slow in LDS): 8 k-values of one column through two transposing reads.
__device__ __forceinline__ bf16x8_t read_b_frag(const unsigned char *tile, int ks, int wave, int lane)
{
    const int grp = lane >> 4, i16 = lane & 15;
    const unsigned char *q = tile + (ks * 16 + 8 * (grp >> 1) + (i16 >> 2)) * S_IN +
                             (wave * 32 + 16 * (grp & 1) + 4 * (i16 & 3)) * 2;
    i16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LBP_LDS_PTR(i16x4_t, q));
    i16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LBP_LDS_PTR(i16x4_t, q + 4 * S_IN));
    return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

}  // namespace lbp
