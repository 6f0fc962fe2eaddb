// Closest centroid of a sub-vector (Section 2.1 of the paper), shared by the encoder and the trainer.
//
// The result is defined by float64 distances: (double)x - (double)c squared and summed in increasing
// component order with separate multiply and add, the lowest index among equal distances.  It is found with
// float32 arithmetic: a wavefront holds 64 sub-vectors, a lane each, and walks over the centroids, whose
// components are the same for all lanes and come through scalar loads.  The float32 distance is within a
// factor 1 +- (dsub + 3) 2^-24 of the float64 one, so unless a second centroid lies within that margin of
// the closest the float32 winner is the float64 winner; the few lanes that see such a pair (about one in
// 10^5 on image descriptors), a value near the end of the float32 range, an infinity or a NaN take the
// float64 loop.
//
// Bound by the vector ALU at two instructions per (centroid, component), and for 16 centroids about as
// long by reading the vectors from HBM.
#pragma once

#include "qadc_common.h"

namespace qadc {

// constant address space: wavefront-uniform reads become scalar loads
typedef const float __attribute__((address_space(4))) uniform_float;

__device__ __forceinline__ uniform_float *uniform_ptr(const float *p)
{
    const uint64_t a = (uint64_t)p;
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)a);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));
    return (uniform_float *)(((uint64_t)hi << 32) | lo);
}

// The definition.  bs: nullptr, or what is subtracted (in float32) from x first.
__device__ __attribute__((noinline)) unsigned nearest_centroid_f64(const float *xs, const float *bs, const float *c, int ksub,
                                                                  int dsub)
{
#pragma clang fp contract(off)
    double best = __builtin_inf();
    unsigned arg = 0;
    for (int i = 0; i < ksub; ++i) {
        double acc = 0.0;
        for (int t = 0; t < dsub; ++t) {
            const float xv = bs ? xs[t] - bs[t] : xs[t];
            const double df = (double)xv - (double)c[i * dsub + t];
            acc += df * df;
        }
        if (acc < best) { best = acc; arg = (unsigned)i; }
    }
    return arg;
}

// Index of the centroid of `cb` [KSUB][dsub] (the same for all lanes) closest to this lane's xs [dsub] (minus
// bs when given).  DS: dsub when it is known to the compiler (xv holds the difference), else 0 (xv is not read).
// Every lane's xs and bs must be readable; lanes with ok = false get an unspecified index below KSUB.
template <int KSUB, int DS>
__device__ __forceinline__ unsigned nearest_centroid(const float *xv, const float *xs, const float *bs, const float *cb,
                                                     int dsub_rt, bool ok)
{
#pragma clang fp contract(off)
    const int dsub = DS ? DS : dsub_rt;
    uniform_float *c = uniform_ptr(cb);
    // b1 <= b2: the two smallest distances seen, as unsigned images (a NaN is above every number).  With 16
    // centroids the index travels in the four low bits of the image.
    constexpr bool PACKED = KSUB == 16;
    unsigned b1 = 0xffffffffu, b2 = 0xffffffffu, arg = 0;
    for (int g = 0; g < KSUB; g += 16) {
        float acc[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = 0.0f;
        uniform_float *cg = c + (size_t)g * dsub;
        if constexpr (DS != 0) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
#pragma unroll
                for (int t = 0; t < DS; ++t) {
                    const float df = xv[t] - cg[i * DS + t];
                    acc[i] = fmaf(df, df, acc[i]);
                }
            }
        } else {
            int t = 0;
            for (; t + 4 <= dsub; t += 4) {
                float x4[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) x4[u] = bs ? xs[t + u] - bs[t + u] : xs[t + u];
#pragma unroll
                for (int i = 0; i < 16; ++i) {
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const float df = x4[u] - cg[i * dsub + t + u];
                        acc[i] = fmaf(df, df, acc[i]);
                    }
                }
            }
            for (; t < dsub; ++t) {
                const float x1 = bs ? xs[t] - bs[t] : xs[t];
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const float df = x1 - cg[i * dsub + t];
                    acc[i] = fmaf(df, df, acc[i]);
                }
            }
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            unsigned key = __float_as_uint(acc[i]);
            if constexpr (PACKED) key = (key & ~15u) | (unsigned)i;
            else arg = key < b1 ? (unsigned)(g + i) : arg;
            b2 = max(min(b1, b2), min(max(b1, b2), key));  // the middle one of the three
            b1 = min(b1, key);
        }
    }
    if constexpr (PACKED) arg = b1 & 15u;
    const float d1 = __uint_as_float(PACKED ? b1 & ~15u : b1), d2 = __uint_as_float(PACKED ? b2 & ~15u : b2);
    // Rounding of both distances, the bits the index took, and results below the normal range.
    const float margin = fmaf(d1, 1e-5f + 3e-7f * (float)dsub, (float)dsub * 1e-36f);
    const bool sure = d1 < 1e37f && d2 > d1 + margin;
    if (ok && !sure) arg = nearest_centroid_f64(xs, bs, cb, KSUB, dsub);
    return arg;
}

}  // namespace qadc
