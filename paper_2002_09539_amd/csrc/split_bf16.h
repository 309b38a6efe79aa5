// fp32 matrix products on the bf16 matrix cores without giving up fp32 accuracy.
//
// Every fp32 operand is split EXACTLY into three bf16 terms, x = hi + mid + lo: hi = bf16(x), mid = bf16(x - hi),
// lo = bf16(x - hi - mid).  A bf16 carries 8 significant bits and each rounding to nearest leaves a remainder of at most
// half a unit of the term before it, so three terms hold the 24 bits of an fp32 (as long as lo stays a normal number:
// |x| >= 2^-109; below that the missing part is under 2^-133 in absolute value: a forward GEMM whose whole batch is of order
// 2^-108 / 2^-112 / 2^-116 / 2^-120, with weights that bring its results back to one, is 5e-8 / 1.4e-7 / 2e-6 / 3e-5 from 64
// bits where the fp32 matrix cores are 1.4e-7).  The product of two split numbers is
// the sum of nine products of bf16 numbers, each exact in fp32; the six largest are formed (hi hi, hi mid, mid hi, mid mid,
// hi lo, lo hi).  The three left out (mid lo, lo mid, lo lo) sum to less than 2^-23.9 of |a b| at worst (a remainder is at
// most 2^-8 of the term before it, and lo at most 2^-17 of the operand) and to 2^-27.4 in the root mean square over normal
// operands, where the rounding of one fp32 product is 2^-24 and 2^-25.2.  Six v_mfma_f32_32x32x16_bf16
// take 192 cycles for 16 contraction indices, eight v_mfma_f32_32x32x2_f32 take 512, and a sum over K indices is rounded
// 6 K / 16 times instead of K times.
//
// Infinities and the few finite numbers that round to a bf16 infinity (|x| >= 0x1.FFp127) take a separate path that
// truncates hi and leaves no remainder behind an infinity; a NaN makes hi a NaN.  The products hi hi then carry the
// infinity or the NaN that fp32 would, but those of an infinity with the other operand's remainders are NaN (a remainder of
// zero) or of either sign, and so are those of finite operands whose product overflows: split_sum leaves the small products
// out where the large ones' sum is not finite.
#pragma once
#include "gemm_bf16_tile.h"

namespace ols {

struct Split8 {
    u4 hi, mid, lo;   // eight bf16 each, in element order
};

__device__ __forceinline__ unsigned pack_bf16(float a, float b) {   // round to nearest even (v_cvt_pk_bf16_f32)
    return __builtin_bit_cast(unsigned, __builtin_convertvector(f2v{a, b}, bf16x2));
}
__device__ __forceinline__ float bf16_lo(unsigned w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(unsigned w) { return __uint_as_float(w & 0xFFFF0000u); }

constexpr float kRoundsToInf = 0x1.FFp127f;

// Eight consecutive elements without the separate path: 44 instructions, and four that keep the largest magnitude in
// `top`.  Where top reaches kRoundsToInf the result is not to be used; callers that split many vectors look once.
__device__ __forceinline__ Split8 split8_finite(f4 a, f4 b, float& top) {
    const float x[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
#pragma unroll
    for (int e = 0; e < 8; e += 2) top = fmaxf(fmaxf(top, fabsf(x[e])), fabsf(x[e + 1]));
    Split8 s;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        s.hi[e] = pack_bf16(x[2 * e], x[2 * e + 1]);
        const float r0 = x[2 * e] - bf16_lo(s.hi[e]), r1 = x[2 * e + 1] - bf16_hi(s.hi[e]);
        s.mid[e] = pack_bf16(r0, r1);
        s.lo[e] = pack_bf16(r0 - bf16_lo(s.mid[e]), r1 - bf16_hi(s.mid[e]));
    }
    return s;
}

// Eight consecutive elements of any value.
__device__ __forceinline__ Split8 split8(f4 a, f4 b) {
    const float x[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
    float top = 0.0f;
    Split8 s = split8_finite(a, b, top);
    if (__builtin_expect(top >= kRoundsToInf, 0)) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float h[2], r[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const float v = x[2 * e + t];
                const bool huge = fabsf(v) >= kRoundsToInf;   // false for a NaN
                h[t] = huge ? __uint_as_float(__float_as_uint(v) & 0xFFFF0000u) : v;
            }
            s.hi[e] = pack_bf16(h[0], h[1]);
            r[0] = __builtin_isinf(x[2 * e]) ? 0.0f : x[2 * e] - bf16_lo(s.hi[e]);
            r[1] = __builtin_isinf(x[2 * e + 1]) ? 0.0f : x[2 * e + 1] - bf16_hi(s.hi[e]);
            s.mid[e] = pack_bf16(r[0], r[1]);
            s.lo[e] = pack_bf16(r[0] - bf16_lo(s.mid[e]), r[1] - bf16_hi(s.mid[e]));
        }
    }
    return s;
}

// The six products of two split fragments.  The five small ones have a sum of their own (`low`), so that the large one is
// rounded against the running sum once per 16 indices and the small ones against a sum 2^-8 of its size.  Gradients of the
// residual block against 64 bits (relative 2-norm per worker, median over 24; 64 channels 32 x 32 / 128 channels 13 x 15 /
// 32 channels 20 x 20): fp32 matrix cores 2.4e-7 / 2.4e-7 / 2.2e-7, one sum for all six products 2.7e-7 / 2.7e-7 /
// 2.6e-7, two sums 1.1e-7 / 1.2e-7 / 1.2e-7.
struct SplitFrag {
    bf16x8 hi, mid, lo;
};
template <int J>
__device__ __forceinline__ void mfma_split(f16v (&acc)[J], f16v (&low)[J], const SplitFrag (&a)[J], const SplitFrag& b) {
#pragma unroll
    for (int j = 0; j < J; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[j].hi, b.hi, acc[j], 0, 0, 0);
#pragma unroll
    for (int j = 0; j < J; ++j) low[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[j].lo, b.hi, low[j], 0, 0, 0);
#pragma unroll
    for (int j = 0; j < J; ++j) low[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[j].hi, b.lo, low[j], 0, 0, 0);
#pragma unroll
    for (int j = 0; j < J; ++j) low[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[j].mid, b.mid, low[j], 0, 0, 0);
#pragma unroll
    for (int j = 0; j < J; ++j) low[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[j].mid, b.hi, low[j], 0, 0, 0);
#pragma unroll
    for (int j = 0; j < J; ++j) low[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[j].hi, b.mid, low[j], 0, 0, 0);
}

// The result of a sum of split products: the large products' sum and the small ones'.
__device__ __forceinline__ float split_sum(float acc, float low) { return __builtin_isfinite(acc) ? acc + low : acc; }

}  // namespace ols
