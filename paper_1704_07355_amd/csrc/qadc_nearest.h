// Closest centroid of a sub-vector (Section 2.1 of the paper), shared by the encoder and the trainer.
//
// The result is defined by float64 distances: (double)x - (double)c squared and summed in increasing
// component order with separate multiply and add, the lowest index among equal distances.  It is found with
// float32 arithmetic: a wavefront holds 64 sub-vectors, a lane each, and walks over the centroids, whose
// components are the same for all lanes and come through scalar loads.  The float32 distance is within a
// factor 1 +- (dsub + 3) 2^-24 of the float64 one, so unless a second centroid lies within that margin of
// the closest the float32 winner is the float64 winner.  A wavefront with a lane that sees such a pair (about one
// lane in 10^5 on image descriptors), a value near the end of the float32 range, an infinity or a NaN walks over the
// centroids once more in float64, in the same way: components that are zero everywhere, repeated centroids and
// integers make that the rule for some data.  500 k vectors of 16 x 8 components, 16 centroids: 56 us, all of them ties
// 174 (in float64 throughout 227; a lane at a time, from memory, the ties took 11,600); 200 k of 8 x 8, 256 centroids:
// 204 and 656 us (8277).  Only ties of 21 to 25 components and 16 centroids are slower than all in float64, by up to 16 %.
//
// Bound by the vector ALU at two instructions per (centroid, component), and for 16 centroids about as
// long by reading the vectors from HBM.
#pragma once

#include <type_traits>

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

// f(x, t, W) for the components t .. t+W-1 of xs (minus bs), W = 8 and then 4, 2, 1: a block's loads travel together.
template <typename F>
__device__ __forceinline__ void component_blocks(const float *xs, const float *bs, int dsub, F f)
{
    int t = 0;
    auto block = [&](auto w) {
        constexpr int W = decltype(w)::value;
        float x[W];
#pragma unroll
        for (int u = 0; u < W; ++u) x[u] = bs ? xs[t + u] - bs[t + u] : xs[t + u];
        f(x, t, w);
        t += W;
    };
    while (t + 8 <= dsub) block(std::integral_constant<int, 8>());
    if (dsub & 4) block(std::integral_constant<int, 4>());
    if (dsub & 2) block(std::integral_constant<int, 2>());
    if (dsub & 1) block(std::integral_constant<int, 1>());
}

// The definition, for a whole wavefront (the centroids come through scalar loads here too).  Arguments as below.
template <int KSUB, int DS>
__device__ __forceinline__ unsigned nearest_centroid_f64(const float *xv, const float *xs, const float *bs, uniform_float *c,
                                                         int dsub)
{
#pragma clang fp contract(off)
    constexpr int N = DS ? 4 : 16;  // centroids side by side
    double best = __builtin_inf();
    unsigned arg = 0;
#pragma unroll 1
    for (int g = 0; g < KSUB; g += N) {
        uniform_float *cg = c + (size_t)g * dsub;
        double acc[N];
#pragma unroll
        for (int i = 0; i < N; ++i) acc[i] = 0.0;
        auto add = [&](float x, int t) {
#pragma clang fp contract(off)
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const double df = (double)x - (double)cg[i * dsub + t];
                acc[i] += df * df;
            }
        };
        if constexpr (DS != 0) {
#pragma unroll
            for (int t = 0; t < DS; ++t) {
                float x = xv[t];
                // (converted anew in every round, one component after the other: side by side the doubles cost the kernel
                // half its wavefronts)
                asm volatile("" : "+v"(x));
                add(x, t);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            component_blocks(xs, bs, dsub, [&](const float *x, int t, auto w) {
#pragma unroll
                for (int u = 0; u < decltype(w)::value; ++u) add(x[u], t + u);
            });
        }
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (acc[i] < best) { best = acc[i]; arg = (unsigned)(g + i); }
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
            component_blocks(xs, bs, dsub, [&](const float *x, int t, auto w) {
#pragma unroll
                for (int i = 0; i < 16; ++i) {
#pragma unroll
                    for (int u = 0; u < decltype(w)::value; ++u) {
                        const float df = x[u] - cg[i * dsub + t + u];
                        acc[i] = fmaf(df, df, acc[i]);
                    }
                }
            });
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
    if (__ballot(ok && !sure) != 0ull) {  // uniform
        const unsigned exact = nearest_centroid_f64<KSUB, DS>(xv, xs, bs, c, dsub);
        if (!sure) arg = exact;
    }
    return arg;
}

}  // namespace qadc
