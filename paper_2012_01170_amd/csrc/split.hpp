// Float32 products on the bf16 matrix cores.
//
// A float32 x is the exact sum of three bf16 values h + m + l (8 + 8 + 8
// significand bits; h is x truncated, so it never overflows; the three-way
// splitting of operands is a published method), and a product x y is the sum of
// the six products hh, hm, mh, mm, hl, lh up to 2^-22 of itself (ml, lm and ll
// are left out: at most 2^-22.02, where both m are near 2^-7 of their operands;
// their mean square is 2^-25).  Each bf16 product is exact in the matrix core's
// float32 accumulation, so over many terms a contraction of split operands is
// closer than one of float32 operands: K 512 of normal values has a relative
// error of 1.4e-7 with the six products summed as below, 4.5e-7 by
// v_mfma_f32_16x16x4_f32 (measured against float64; K 1024: 1.7e-7 and 5.8e-7).
//
// What the split loses are tiny operands.  bf16 reaches down to 2^-133, so an
// operand below 2^-110 keeps multiples of that only: a relative error of up to
// 2^-134 / |x|, 2^-20 at 2^-114 (5e-35) and 2^-10 at 2^-124 (measured: 3e-7 and
// 3e-4), where a float32 product still has 2^-24.
//
// Six 16x16x32 bf16 instructions take 96 cycles where eight 16x16x4 float32 ones
// take 256 for the same products; what the pass gains from that is less, since
// the gather and the split run beside it (tile_kernels.hpp has its times).
//
// The leading products hh are summed apart from the five others (hi and lo):
// the small terms then keep their low bits, and an infinity or NaN among the
// operands, whose m and l are NaN, gives what it gives in float32 (finish();
// a NaN has to be a quiet one, see quiet()).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace sbc {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));

// two float32 -> two bf16 (nearest even) in one word, a in the low half
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    typedef float f2 __attribute__((ext_vector_type(2)));
    typedef __bf16 b2 __attribute__((ext_vector_type(2)));
    const f2 v{a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, b2));
}

// x, a NaN with bit 22 set: the upper half of one whose payload lies in the
// lower half alone reads as an infinity.  For operands as they lie in memory
// (what arithmetic makes of a NaN has the bit).
__device__ __forceinline__ float quiet(float x) {
    return x == x ? x : __uint_as_float(__float_as_uint(x) | 0x00400000u);
}

// (a, b) -> their h, m and l parts, each as a word with a in the low half
__device__ __forceinline__ void split2(float a, float b, uint32_t &h, uint32_t &m, uint32_t &l) {
    const uint32_t ua = __float_as_uint(a), ub = __float_as_uint(b);
    h = __builtin_amdgcn_perm(ub, ua, 0x07060302u);  // the upper halves
    const float ra = a - __uint_as_float(ua & 0xFFFF0000u);
    const float rb = b - __uint_as_float(ub & 0xFFFF0000u);
    m = pack_bf16(ra, rb);
    l = pack_bf16(ra - __uint_as_float(m << 16), rb - __uint_as_float(m & 0xFFFF0000u));
}

// The products of one k-step of operands a and b of NA and NB parts (3, or 1
// for a bf16 operand, which is its own h), smallest first.
template <int NA, int NB>
__device__ __forceinline__ void mma_split(const bf16x8 (&a)[NA], const bf16x8 (&b)[NB],
                                          floatx4 &hi, floatx4 &lo) {
    static_assert((NA == 3 || NA == 1) && (NB == 3 || NB == 1), "parts");
#define SBC_MMA(x, y, acc) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[x], b[y], acc, 0, 0, 0)
    if constexpr (NA == 3) SBC_MMA(NA - 1, 0, lo);
    if constexpr (NB == 3) SBC_MMA(0, NB - 1, lo);
    if constexpr (NA == 3 && NB == 3) SBC_MMA(NA / 2, NB / 2, lo);
    if constexpr (NA == 3) SBC_MMA(NA / 2, 0, lo);
    if constexpr (NB == 3) SBC_MMA(0, NB / 2, lo);
    SBC_MMA(0, 0, hi);
#undef SBC_MMA
}

// hi + lo; a non-finite hi stands for itself (lo, of which an infinite operand
// makes NaN, is left out then)
__device__ __forceinline__ float finish(float hi, float lo) {
    const float s = hi + lo;
    return s == s ? s : hi;
}

__device__ __forceinline__ floatx4 finish(const floatx4 &hi, const floatx4 &lo) {
    return floatx4{finish(hi[0], lo[0]), finish(hi[1], lo[1]), finish(hi[2], lo[2]),
                   finish(hi[3], lo[3])};
}

}  // namespace sbc
