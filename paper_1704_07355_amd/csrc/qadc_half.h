// Products of binary16 factors as a filter (qadc_assign.hip, qadc_ivf_filter.hip): x' and c', the differences of a vector
// and of a centroid to a reference vector, scaled by a power of two, are rounded to binary16 and multiplied by the matrix
// units; score = |c'|^2 - 2 x^.c^ is distance^2 - |x'|^2 up to a rounding that is bounded here.
#pragma once

#include "qadc_common.h"

namespace qadc {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef unsigned bits16x8 __attribute__((ext_vector_type(4)));  // eight 16-bit numbers of either kind
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Eight consecutive components t .. t+7 of a row, zero at and beyond d.  VEC: 16-byte aligned rows of whole steps.  Other
// rows: whole eights in wide loads (a test per component otherwise: 1 M vectors, K = 256, d = 100 1.00 -> 0.80, d = 40 0.82 ->
// 0.65 of the time), the rest one by one.  SKIP: no look at eights beyond d -- worth its branch where a row has many of them or
// the registers for them are short (d = 136 to 250: 1.05 -> 0.90), not otherwise (d = 8, 1 M vectors 0.97 -> 1.14).
template <bool VEC, bool SKIP = false>
__device__ __forceinline__ f32x8 load8(const float *row, int t, int d)
{
    f32x8 v;
    if constexpr (VEC) {
        const float4 a = *reinterpret_cast<const float4 *>(row + t);
        const float4 b = *reinterpret_cast<const float4 *>(row + t + 4);
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
        v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    } else if constexpr (SKIP) {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = 0.0f;
        if (t + 8 <= d) {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = row[t + e];
        } else if (t < d) {
#pragma unroll
            for (int e = 0; e < 7; ++e) {
                const float f = row[min(t + e, d - 1)];
                v[e] = t + e < d ? f : 0.0f;
            }
        }
    } else if (t + 8 <= d) {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = row[t + e];
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = t + e < d ? row[t + e] : 0.0f;
    }
    return v;
}

// Component t of the reference: the middle of eight centroids of the range.  (Any vector would do; one amid the centroids
// keeps the norms, and with them the margins, small, and a few stray or non-finite ones do not move this.)  *spread becomes
// at least how far those centroids are from it, but for one at either end.
__device__ __forceinline__ float reference_component(const float *__restrict__ coarse, int K, int d, int t, float *spread)
{
    float v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = t < d ? coarse[(size_t)((int64_t)k * K >> 3) * d + t] : 0.0f;
#pragma unroll
    for (int a = 0; a < 8; ++a)  // odd-even transposition sort (a NaN goes out at the first comparison)
#pragma unroll
        for (int b = a & 1; b + 1 < 8; b += 2) {
            const float lo = fminf(v[b], v[b + 1]), hi = fmaxf(v[b], v[b + 1]);
            v[b] = lo;
            v[b + 1] = hi;
        }
    const float ref = 0.5f * v[3] + 0.5f * v[4];
    const float f = fmaxf(v[6] - ref, ref - v[1]);
    if (f < 3e38f) *spread = fmaxf(*spread, f);
    return ref;
}

// The power of two that takes the spread to 16 .. 32: a thousandth of that still has eleven bits, two thousand times as much
// is still in range.
__device__ __forceinline__ float half_scale(float spread)
{
    const int e = (int)(__float_as_uint(spread) >> 23) - 127;  // (-127: nothing at all, or less than 2^-126)
    return __uint_as_float((unsigned)(127 + min(100, 4 - e)) << 23);
}

// |score - (distance^2 - |x'|^2)| <= xerr + cerr, of components in D: the conversions leave ex = |x' - x^| and ec = |c' - c^| <= 2^-11 |c'|; 2 |x^.c^ - x'.c'| <= 2 ex |c^| + 2 |x'| ec,
// and with 2 a b <= w a^2 + b^2 / w that is 2^12 ex^2 + 2^-11 |x'|^2 of the vector (ex is measured, mostly 0.4 2^-11 |x'|)
// and (2^-12 + 2^-11) |c'|^2 of the centroid (ec is not: that would be two fifths of the conversion's work).  Should the
// units take what is below the normal range, 2^-14, for zero: (e + 2^-14 sqrt D)^2 <= 17/16 e^2 + 17 D 2^-28, which is
// HALF_CONV and HALF_TINY and a sixteenth on ec^2.  With the differences, D + 1 additions and the norms (1e-6 + 3.0e-7 D
// of the square) 4.9e-4 + 3.0e-7 D of the vector's and 7.7e-4 + 3.0e-7 D of the centroid's.
// xerr = half_eps(D) |x'|^2 + HALF_CONV ex^2 + HALF_TINY D, cerr = half_eps_c(D) |c'|^2 + HALF_TINY D; each D + 1 additions of
// values up to 2 (|x'|^2 + |c'|^2) at 2^-23, no assumption on how the matrix units round.
constexpr float half_eps(int D) { return 5.1e-4f + 3.3e-7f * (float)D; }
constexpr float half_eps_c(int D) { return 7.9e-4f + 3.3e-7f * (float)D; }
// The bound holds for scores up to HALF_FAR, of vectors with |x'|^2 up to HALF_NEAR.  A centroid with |c'|^2 beyond HALF_STRAY
// may not fit binary16: 0.29 |c'|^2 is no more than |c'|^2 - 2 x'.c' of any such vector, and stands for its score.
constexpr float HALF_NEAR = 268435456.0f;   // 2^28
constexpr float HALF_STRAY = 2147483648.0f; // 2^31: no component of a centroid below it leaves binary16
constexpr float HALF_FAR = 5e8f;
constexpr float HALF_CONV = 4400.0f;        // 2^12, and a sixteenth for what HALF_TINY pays for
constexpr float HALF_TINY = 3e-4f;          // per component: conversions below the normal range of binary16, flushed or not

}  // namespace qadc
