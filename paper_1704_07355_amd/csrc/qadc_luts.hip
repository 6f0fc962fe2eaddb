// Tables step (Eq. (1) of the paper) and 8-bit quantization of the tables
// (Section 3.3) on gfx950.  Both are tiny next to the scan, and bound by the latency of their steps.

#include <algorithm>

#include "qadc_scan_common.h"

namespace qadc {

// ------------------------------------------------------------------ Eq. (1)

// luts[q][j][i] = sum_t (y[q][j*dsub+t] - base[q][j*dsub+t] - C[j][i][t])^2.
// Differences and the sum are taken in float64 and rounded once to float32, so
// a residual query (y - base) loses nothing to an intermediate rounding.
// A workgroup per query, the query's differences in LDS, walks over the entries.
__global__ __launch_bounds__(256) void build_luts_kernel(
    const float *__restrict__ codebooks, int d, int m, int ksub, const float *__restrict__ queries,
    const float *__restrict__ base, float *__restrict__ luts)
{
    extern __shared__ double yq[];  // [d]
    const int q = blockIdx.x;
    const int dsub = d / m;
    for (int t = threadIdx.x; t < d; t += 256) {
        double y = (double)queries[(size_t)q * d + t];
        if (base) y -= (double)base[(size_t)q * d + t];
        yq[t] = y;
    }
    __syncthreads();
    const int entries = m * ksub;
    for (int e = threadIdx.x; e < entries; e += 256) {
        const float *c = codebooks + (size_t)e * dsub;
        const double *y = yq + e / ksub * dsub;
        double acc = 0.0;
        for (int t = 0; t < dsub; ++t) {
            const double df = y[t] - (double)c[t];
            acc += df * df;
        }
        luts[(size_t)q * entries + e] = (float)acc;
    }
}

// The same entries, a thread for each and a workgroup per 256 of them; eight components are requested at a time.
__global__ __launch_bounds__(256) void build_luts_wide_kernel(
    const float *__restrict__ codebooks, int d, int m, int ksub, const float *__restrict__ queries,
    const float *__restrict__ base, float *__restrict__ luts)
{
    const int q = blockIdx.y;
    const int dsub = d / m;
    const int entries = m * ksub;
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= entries) return;
    const float *c = codebooks + (size_t)e * dsub;
    const size_t at = (size_t)q * d + (size_t)(e / ksub) * dsub;
    double acc = 0.0;
    for (int t0 = 0; t0 < dsub; t0 += 8) {
        float cv[8], yv[8], bv[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const int tt = min(t0 + t, dsub - 1);
            cv[t] = c[tt];
            yv[t] = queries[at + tt];
            bv[t] = base ? base[at + tt] : 0.0f;
        }
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            if (t0 + t < dsub) {
                double y = (double)yv[t];
                if (base) y -= (double)bv[t];
                const double df = y - (double)cv[t];
                acc += df * df;
            }
        }
    }
    luts[(size_t)q * entries + e] = (float)acc;
}

// A few queries of 2048 entries and more: eight rounds and more of one workgroup, each a round trip, against one (us, a workgroup
// per query / a thread per entry: 1 query of 8 x 256 entries of 12 components 6.8 / 4.6, of 120 22 / 16, 64 of 32 x 256 of 4
// 16.9 / 6.4, 128 17.8 / 11.2).  More queries: a thread per entry reads the query again for every entry and twice the lines of
// the codebook (8 x 256 of 12: 64 queries 6.7 / 4.2, 128 6.8 / 6.1, 256 7.5 / 10.3, 4096 50 / 135; of 120: 16 22 / 17, 33 23 / 30,
// 512 44 / 327; 32 x 64 of 8: 64 4.2 / 4.4, 256 5.2 / 9.5).
static bool luts_wide_pay(int d, int m, int ksub, int nq)
{
    const int64_t entries = (int64_t)m * ksub, dsub = d / m;
    return entries >= 2048 && ceil_div(entries, 256) * nq * dsub <= (entries >= 8192 || dsub >= 64 ? 16384 : 8192);
}

int build_luts(const float *codebooks, int d, int m, int ksub, const float *queries,
               const float *base, int nq, float *luts, hipStream_t st)
{
    if (!codebooks || !queries || !luts) return fail(QADC_EINVAL, "qadc_build_luts: null pointer");
    if (m < 1 || d < m || d % m != 0 || (ksub != 16 && ksub != 64 && ksub != 256) || nq < 0 || d > 8192)
        return fail(QADC_EINVAL, "qadc_build_luts: unsupported d=%d m=%d ksub=%d nq=%d", d, m, ksub, nq);
    if (nq == 0) return QADC_OK;
    if (luts_wide_pay(d, m, ksub, nq))  // (at most 2048 queries)
        launch(QADC_PROF_TABLES, build_luts_wide_kernel, dim3((unsigned)ceil_div((int64_t)m * ksub, 256), (unsigned)nq), dim3(256), 0,
               st, codebooks, d, m, ksub, queries, base, luts);
    else
        launch(QADC_PROF_TABLES, build_luts_kernel, dim3((unsigned)nq), dim3(256), (size_t)d * sizeof(double), st, codebooks, d, m,
               ksub, queries, base, luts);
    QADC_HIP_TRY(hipGetLastError());
    return QADC_OK;
}

// -------------------------------------------------------------- Section 3.3

constexpr int QUANT_NT = 1024;

// KSUB = 16: 4-bit components, two per code byte (the paper's case).  KSUB = 256: 8-bit components,
// one per code byte, the same quantizer applied to the 256-entry tables of Section 2.1's
// standard product quantizer.  KSUB = 64: 6-bit components (the paper's Conclusion), stored back to
// back, least significant bit first, four per three bytes.

// The bytes of a code (from any address) as words, all requested at once.
template <int B>
__device__ __forceinline__ void code_words(const uint8_t *c, unsigned (&w)[(B + 3) / 4])
{
    if constexpr (B % 4 != 0) w[B / 4] = 0;
    __builtin_memcpy(w, c, B);
}

// Float ADC sum of a code (Eq. (2), float32, increasing component) over tables of KSUB entries.
template <int KSUB, int B>
__device__ __forceinline__ float sum_of_code(const unsigned (&w)[(B + 3) / 4], const float *lut)
{
    float acc = 0.0f;
    if constexpr (KSUB == 64) {
#pragma unroll
        for (int j = 0; j < 4 * B / 3; ++j) {
            const int k = 6 * j >> 5, sh = 6 * j & 31;
            const unsigned v = sh <= 26 ? w[k] >> sh : __funnelshift_r(w[k], w[min(k + 1, (B - 1) / 4)], sh);
            acc = acc + lut[j * 64 + (v & 63u)];
        }
    } else {
#pragma unroll
        for (int jb = 0; jb < B; ++jb) {
            const unsigned comps = (w[jb >> 2] >> (8 * (jb & 3))) & 0xffu;
            if constexpr (KSUB == 16) {
                acc = acc + lut[(2 * jb) * 16 + (comps & 15u)];
                acc = acc + lut[(2 * jb + 1) * 16 + (comps >> 4)];
            } else {
                acc = acc + lut[jb * 256 + comps];
            }
        }
    }
    return acc;
}

// The need-th smallest of n images of sums in LDS, by the whole workgroup.  (As a call, which the compiler makes of it
// by itself, 1 to 3 us more for some thousand sums.)
__device__ __forceinline__ unsigned nth_of_sums(const unsigned *cand, int n, int need, SelectScratch *sc)
{
    unsigned nth;
    [[clang::always_inline]] nth = block_radix_select_each<unsigned, 4>(
        [&](auto f) {
            for (unsigned i = threadIdx.x; i < (unsigned)n; i += blockDim.x) f(cand[i]);
        },
        (unsigned)need, sc);
    return nth;
}

// A workgroup per query, two per compute unit (64 registers).  Bound by the chain of its steps for a few queries, by the
// instructions of the sums and the selection for thousands.  One form per length of a code: with the number of words a number at
// run time, each word behind a branch, a code's sum took twice as long (us; 4096 queries, 200 init codes, m = 16 84 -> 39, 8000
// of m = 64 637 -> 267, one query 41 -> 28; 1000 queries, 200 codes of 32 six-bit components 44 -> 21).
template <int KSUB, int B>
__global__ __launch_bounds__(QUANT_NT, 8) void quantize_luts_kernel(
    const float *__restrict__ luts, int ngroup, const uint8_t *__restrict__ init_codes,
    int n_init, const float *__restrict__ qmax_in, int R, int nbins, int qmin_mode,
    uint8_t *__restrict__ qluts, float *__restrict__ bias_out, float *__restrict__ delta_out,
    float *__restrict__ qmax_out)
{
    constexpr int m = KSUB == 16 ? 2 * B : KSUB == 64 ? 4 * B / 3 : B;
    __shared__ float lut0[KSUB == 16 ? m * 16 : 1];
    __shared__ unsigned cand[QADC_MAX_INIT];
    __shared__ unsigned bias_ord[m];
    __shared__ float bias[m];
    __shared__ float delta_s;
    __shared__ SelectScratch sc;

    const int tid = threadIdx.x;
    const int q = blockIdx.x;
    constexpr int LOG = KSUB == 16 ? 4 : KSUB == 64 ? 6 : 8;
    constexpr int entries = m * KSUB;
    const float *lq = luts + (size_t)q * ngroup * entries;

    if (KSUB == 16)
        for (int e = tid; e < entries; e += QUANT_NT) lut0[e] = lq[e];
    for (int j = tid; j < m; j += QUANT_NT) bias_ord[j] = 0xffffffffu;
    __syncthreads();

    // qmax: R-th smallest float ADC distance of the init codes, with the first table set (cached after the first touch)
    float qmax;
    if (init_codes) {
        for (int i = tid; i < n_init; i += QUANT_NT) {
            unsigned w[(B + 3) / 4];
            code_words<B>(init_codes + (size_t)i * B, w);
            cand[i] = f2ord(sum_of_code<KSUB, B>(w, KSUB == 16 ? lut0 : lq));
        }
        __syncthreads();
        qmax = ord2f(nth_of_sums(cand, n_init, min(R, n_init), &sc));
    } else {
        qmax = qmax_in[q];
    }

    // bias_j = minimum of table j over every table set of the query.  A thread meets the same
    // table positions in every set (entries and the thread count divide one another): minimum in
    // a register first, one LDS atomic per position.
    if (entries >= QUANT_NT) {
        for (int pos = tid; pos < entries; pos += QUANT_NT) {
            unsigned mn = 0xffffffffu;
#pragma unroll 8
            for (int g = 0; g < ngroup; ++g) mn = min(mn, f2ord(lq[(size_t)g * entries + pos]));
            atomicMin(&bias_ord[pos >> LOG], mn);
        }
    } else {
        const int pos = tid % entries;
        unsigned mn = 0xffffffffu;
#pragma unroll 8
        for (int g = tid / entries; g < ngroup; g += QUANT_NT / entries)
            mn = min(mn, f2ord(lq[(size_t)g * entries + pos]));
        atomicMin(&bias_ord[pos >> LOG], mn);
    }
    __syncthreads();
    for (int j = tid; j < m; j += QUANT_NT) bias[j] = ord2f(bias_ord[j]);
    __syncthreads();
    if (tid == 0) {
        float qmin;
        if (qmin_mode == QADC_QMIN_GLOBAL) {
            unsigned g = 0xffffffffu;
            for (int j = 0; j < m; ++j) g = min(g, bias_ord[j]);
            qmin = ord2f(g);
            for (int j = 0; j < m; ++j) bias[j] = qmin;
        } else {
            qmin = 0.0f;
#pragma unroll 8
            for (int j = 0; j < m; ++j) qmin = qmin + bias[j];
        }
        float delta = __fdiv_rn(qmax - qmin, (float)nbins);
        if (!(delta > 0.0f)) delta = 1.0f;
        delta_s = delta;
        if (delta_out) delta_out[q] = delta;
        if (qmax_out) qmax_out[q] = qmax;
    }
    __syncthreads();
    const float delta = delta_s;
    if (bias_out)
        for (int j = tid; j < m; j += QUANT_NT) bias_out[(size_t)q * m + j] = bias[j];

    const float top = (float)nbins;
    uint8_t *qq = qluts + (size_t)q * ngroup * entries;
#pragma unroll 4
    for (int e = tid; e < ngroup * entries; e += QUANT_NT) {
        const float off = fmaxf(0.0f, lq[e] - bias[(e % entries) >> LOG]);
        const float t = floorf(__fdiv_rn(off, delta));
        qq[e] = (t < top) ? (uint8_t)t : (uint8_t)nbins;
    }
}

int quantize_luts(int ksub, const float *luts, int nq, int ngroup, int m, const uint8_t *init_codes,
                  int64_t n_init, const float *qmax_in, int R, int nbins, int qmin_mode,
                  uint8_t *qluts, float *bias, float *delta, float *qmax_out, hipStream_t st)
{
    if (!luts || !qluts) return fail(QADC_EINVAL, "qadc_quantize_luts: null pointer");
    const int mm = ksub == 256 ? 2 * m : m;  // 8-bit components: m in {4, 8, 16, 32}
    if (!(mm == 8 || mm == 16 || mm == 32 || (mm == 64 && ksub != 64)) || nq < 0 || ngroup < 1)
        return fail(QADC_EINVAL, "qadc_quantize_luts: unsupported m=%d nq=%d ngroup=%d", m, nq, ngroup);
    if (nbins < 1 || nbins > 255 || R < 1)
        return fail(QADC_EINVAL, "qadc_quantize_luts: nbins=%d R=%d", nbins, R);
    if (qmin_mode != QADC_QMIN_PER_TABLE && qmin_mode != QADC_QMIN_GLOBAL)
        return fail(QADC_EINVAL, "qadc_quantize_luts: qmin_mode=%d", qmin_mode);
    if (init_codes) {
        if (n_init < 1 || n_init > QADC_MAX_INIT)
            return fail(QADC_EINVAL, "qadc_quantize_luts: n_init=%lld not in 1..%d", (long long)n_init,
                        QADC_MAX_INIT);
    } else if (!qmax_in) {
        return fail(QADC_EINVAL, "qadc_quantize_luts: neither init_codes nor qmax_in given");
    }
    if (nq == 0) return QADC_OK;
#define QADC_QUANT_CASE(KSUB_, B_)                                                                                     \
    case B_:                                                                                                        \
        launch(QADC_PROF_QUANTIZE, quantize_luts_kernel<KSUB_, B_>, dim3(nq), dim3(QUANT_NT), 0, st, luts, ngroup,     \
               init_codes, (int)n_init, qmax_in, R, nbins, qmin_mode, qluts, bias, delta, qmax_out);                \
        break;
    if (ksub == 16) {
        switch (m / 2) {
            QADC_QUANT_CASE(16, 4)
            QADC_QUANT_CASE(16, 8)
            QADC_QUANT_CASE(16, 16)
            QADC_QUANT_CASE(16, 32)
        }
    } else if (ksub == 64) {
        switch (3 * m / 4) {
            QADC_QUANT_CASE(64, 6)
            QADC_QUANT_CASE(64, 12)
            QADC_QUANT_CASE(64, 24)
        }
    } else {
        switch (m) {
            QADC_QUANT_CASE(256, 4)
            QADC_QUANT_CASE(256, 8)
            QADC_QUANT_CASE(256, 16)
            QADC_QUANT_CASE(256, 32)
        }
    }
#undef QADC_QUANT_CASE
    QADC_HIP_TRY(hipGetLastError());
    return QADC_OK;
}

// Both steps for a batch of qadc_search, a workgroup per query and a thread per entry: the float tables stay in LDS and
// are not written.  The arithmetic of build_luts_kernel and quantize_luts_kernel.  (As two launches 9.9 us for 16 queries
// m = 16, 16.1 for 12 m = 64; 8.9 and 12.1 as one; 500 queries, 8000 init codes, m = 64 51.6, 83.7 with the sum's loop over a number
// of words that the compiler does not know.)
constexpr int SEARCH_TABLES_MAX_D = 2048;

template <int B>
__global__ __launch_bounds__(1024, 8) void search_tables_kernel(
    const float *__restrict__ codebooks, int d, const float *__restrict__ queries, const uint8_t *__restrict__ codes,
    int n_init, int R, int nbins, int qmin_mode, uint8_t *__restrict__ qluts, uint8_t *__restrict__ qluts_too,
    float *__restrict__ deltas)
{
    constexpr int m = 2 * B;
    __shared__ float yq[SEARCH_TABLES_MAX_D];
    __shared__ float lut[m * 16];
    __shared__ unsigned cand[QADC_MAX_INIT];
    __shared__ unsigned bias_ord[m];
    __shared__ float bias[m];
    __shared__ float delta_s;
    __shared__ SelectScratch sc;
    constexpr int DREG = 16;
    const int tid = threadIdx.x, q = blockIdx.x;
    constexpr int entries = m * 16;
    const int dsub = d / m;
    // everything that comes from memory is requested at once
    for (int t = tid; t < d; t += 1024) yq[t] = queries[(size_t)q * d + t];
    float cv[DREG];
    const float *c = codebooks + (size_t)min(tid, entries - 1) * dsub;
#pragma unroll
    for (int t = 0; t < DREG; ++t) cv[t] = c[min(t, dsub - 1)];
    unsigned w[B / 4];
    code_words<B>(codes + (size_t)min(tid, n_init - 1) * B, w);
    __syncthreads();
    const int j = tid >> 4;
    float v = 0.0f;
    if (tid < entries) {
        double acc = 0.0;
#pragma unroll
        for (int t = 0; t < DREG; ++t) {
            if (t < dsub) {  // uniform
                const double df = (double)yq[j * dsub + t] - (double)cv[t];
                acc += df * df;
            }
        }
        for (int t = DREG; t < dsub; ++t) {
            const double df = (double)yq[j * dsub + t] - (double)c[t];
            acc += df * df;
        }
        v = (float)acc;
        lut[tid] = v;
        unsigned least = f2ord(v);
#pragma unroll
        for (int k = 8; k >= 1; k >>= 1) least = min(least, (unsigned)__shfl_xor((int)least, k));
        if ((tid & 15) == 0) { bias_ord[j] = least; bias[j] = ord2f(least); }
    }
    __syncthreads();
    for (int i = tid; i < n_init; i += 1024) {
        if (i != tid) code_words<B>(codes + (size_t)i * B, w);
        cand[i] = f2ord(sum_of_code<16, B>(w, lut));
    }
    __syncthreads();
    const float qmax = ord2f(nth_of_sums(cand, n_init, min(R, n_init), &sc));
    if (tid == 0) {
        float qmin;
        if (qmin_mode == QADC_QMIN_GLOBAL) {
            unsigned g = 0xffffffffu;
            for (int k = 0; k < m; ++k) g = min(g, bias_ord[k]);
            qmin = ord2f(g);
            for (int k = 0; k < m; ++k) bias[k] = qmin;
        } else {
            qmin = 0.0f;
#pragma unroll 8
            for (int k = 0; k < m; ++k) qmin = qmin + bias[k];
        }
        float delta = __fdiv_rn(qmax - qmin, (float)nbins);
        if (!(delta > 0.0f)) delta = 1.0f;
        delta_s = delta;
        if (deltas) deltas[q] = delta;
    }
    __syncthreads();
    if (tid < entries) {
        const float t = floorf(__fdiv_rn(fmaxf(0.0f, v - bias[j]), delta_s));
        const uint8_t e = (t < (float)nbins) ? (uint8_t)t : (uint8_t)nbins;
        qluts[(size_t)q * entries + tid] = e;
        if (qluts_too) qluts_too[(size_t)q * entries + tid] = e;
    }
}

void search_tables(const float *codebooks, int d, int m, const float *queries, int nq, const uint8_t *codes, int n_init,
                   int R, int nbins, int qmin_mode, uint8_t *qluts, uint8_t *qluts_too, float *deltas, hipStream_t st)
{
#define QADC_CASE(B_)                                                                                               \
    case B_:                                                                                                        \
        launch(QADC_PROF_TABLES, search_tables_kernel<B_>, dim3((unsigned)nq), dim3(1024), 0, st, codebooks, d, queries, \
               codes, n_init, R, nbins, qmin_mode, qluts, qluts_too, deltas);                                            \
        break;
    switch (m / 2) {
        QADC_CASE(4)
        QADC_CASE(8)
        QADC_CASE(16)
        QADC_CASE(32)
    }
#undef QADC_CASE
}

}  // namespace qadc
