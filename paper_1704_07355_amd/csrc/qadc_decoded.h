// A batch's sums as products of decoded codes: the pieces of scan_u8_decoded_kernel (qadc_scan_decoded.hip).
//
// A quantized table is floor((|y_j - C_j[c]|^2 - bias_j) / Delta), so a code's sum is, up to the floors, an affine function of
// y . x with x the code's decoded vector: a product of d numbers per (code, query) where the exact sum is one of 16 m.  Here both
// factors are rounded to int8 and the product gives a LOWER BOUND of the quantized sum; the pairs it lets pass (some 3e-4, where
// 1e-6 are results) are summed exactly from the quantized tables.  Sums and results are the definition's.
//
// The bound needs no estimate of any rounding.  With whole numbers phi_j[c] (the centroids of table j, in int8), yhat_j (the
// query, in int8) and a whole S > 0,
//     a_j = min over c of  4 S q_j[c] - phi_j[c]^2 + 4 yhat_j . phi_j[c]
// is computed in integers from the quantized entries q_j[c] as they are, whatever they and the roundings are, and then for every code
//     4 S sum q_j[c_j]  >=  sum (phi_j[c_j]^2 - 4 yhat_j . phi_j[c_j]) + sum a_j .
// An entry at the quantizer's last value is left out of the minimum: a code with one has a sum no bound below that value lets pass.
// With n = floor(sum phi^2 / 4), which goes into the accumulator, a sum within `bound` (below the last value) has
//     n - sum yhat . phi  <=  S bound - floor(sum a_j / 4) .
// Scales: phi in units of s, the largest distance of a centroid's component from the middle of its table's / 127; yhat in units
// of 2 s (queries lie further out than centroids; beyond 127 units they are clamped, which only loosens their a_j); S the whole
// number next to Delta / 4 s^2, up to DECODED_MAX_S, so that none of the sums leaves 32 bits.
#pragma once

#include "qadc_onehot.h"

namespace qadc {

constexpr int DECODED_MAX_S = 16384;  // 64 tables x 4 S 255 + what the products add: below 2^31
constexpr int DECODED_NONE = -(1 << 30);  // below every result, and their difference is still 32 bits

// Lookups of decoded components: table t = 2 (code byte) + (high nibble), 16 entries of four int8 each (components beyond
// d / m are zero).  The K = 8 B components of a code of B bytes are taken 32 at a time, one code word: lanes 0..31 (half 0) of
// the operand hold the low nibbles' tables of its four bytes, lanes 32..63 the high ones', 16 bytes per lane either way.
//
// Every byte of the result: offset of the nibble's entry in the 128 bytes of a code byte's two tables.
__device__ __forceinline__ unsigned decoded_offsets(unsigned w, int half)
{
    return (__builtin_amdgcn_alignbit(w, w, half ? 2u : 30u) & 0x3c3c3c3cu) | (half ? 0x40404040u : 0u);
}

// Four components of four tables each: the operand of one matrix instruction.
__device__ __forceinline__ v4i_t decoded_lookup(const int *tab, unsigned w, int word, int half)
{
    const unsigned x = decoded_offsets(w, half);
    const char *t = reinterpret_cast<const char *>(tab) + word * 512;
    v4i_t a;
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = *reinterpret_cast<const int *>(t + i * 128 + __builtin_amdgcn_ubfe(x, 8 * i, 8));
    return a;
}

// How far the components of a codebook lie from the middles of their tables, / 127; mid: the middles of this thread's table.
// Thread = (table, centroid), NT threads; wmax: a word of LDS per wavefront; a barrier inside.
template <int NT>
__device__ __forceinline__ float decoded_scale(const float (&cv)[4], float (&mid)[4], float *wmax)
{
    float far = 0.0f;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        float lo = cv[t], hi = cv[t];
#pragma unroll
        for (int s = 8; s >= 1; s >>= 1) {
            lo = fminf(lo, __shfl_xor(lo, s));
            hi = fmaxf(hi, __shfl_xor(hi, s));
        }
        mid[t] = 0.5f * lo + 0.5f * hi;
        far = fmaxf(far, fmaxf(hi - mid[t], mid[t] - lo));
    }
#pragma unroll
    for (int s = 32; s >= 16; s >>= 1) far = fmaxf(far, __shfl_xor(far, s));
    if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = far;
    __syncthreads();
    for (int k = 0; k < NT / WAVE; ++k) far = fmaxf(far, wmax[k]);
    return far > 1e-30f && far < 1e30f ? far / 127.0f : 1.0f;  // (anything will do: it is only a loose bound then)
}

__device__ __forceinline__ int decoded_steps(float delta, float s)
{
    return (int)fminf(fmaxf(rintf(delta / (4.0f * s * s)), 1.0f), (float)DECODED_MAX_S);  // (a NaN: 1)
}

// a_j of this thread's table, in its 16 lanes (INT32_MAX: every entry is the last value), with its centroid's phi and the
// query's yhat, negated, as four bytes each.
__device__ __forceinline__ int decoded_slack(const float (&cv)[4], const float (&mid)[4], const float (&yv)[4], float s, int S,
                                             int entry, int last, int *phi, int *yhat)
{
    int squares = 0, product = 0;
    unsigned p = 0, y = 0;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int f = (int)fminf(fmaxf(rintf((cv[t] - mid[t]) / s), -127.0f), 127.0f);
        const int h = (int)fminf(fmaxf(rintf((yv[t] - mid[t]) / (2.0f * s)), -127.0f), 127.0f);
        squares += f * f;
        product += f * h;
        p |= (unsigned)(f & 255) << (8 * t);
        y |= (unsigned)(-h & 255) << (8 * t);
    }
    *phi = (int)p;
    *yhat = (int)y;
    int a = entry >= last ? INT32_MAX : 4 * S * entry - squares + 4 * product;
#pragma unroll
    for (int k = 8; k >= 1; k >>= 1) a = min(a, __shfl_xor(a, k));
    return a;
}

// Exact sum of a code (words w[]) over a query's quantized tables [2 B][16].
template <int B>
__device__ __forceinline__ unsigned exact_sum(const uint8_t *ql, const unsigned (&w)[B / 4])
{
    unsigned sum = 0;
#pragma unroll
    for (int jb = 0; jb < B; ++jb) {
        const unsigned c = __builtin_amdgcn_ubfe(w[jb >> 2], 8 * (jb & 3), 8);
        sum += (unsigned)ql[32 * jb + (c & 15u)] + (unsigned)ql[32 * jb + 16 + (c >> 4)];
    }
    return sum;
}

}  // namespace qadc
