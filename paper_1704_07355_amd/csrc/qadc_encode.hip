// Database side of product quantization on gfx950 (Section 2.1 of the paper):
// enc(x) = (i_0 .. i_{m-1}), i_j = argmin_i || x^j - C^j[i] ||^2, written in the
// standard code layout; for an inverted index (Section 2.2) the vector encoded at storage
// position p is the residual x[ids[p]] - coarse[cells[ids[p]]].  Not on the query path.

#include "qadc_nearest.h"

namespace qadc {

// Where the centroids of the cells come from: a table of K rows, or the two half-quantizers of a
// multi-index (cell c = i*Kh + j, centroid (halves[0][i], halves[1][j]); with m even a sub-vector
// lies inside one half).  `off` = first dimension of the sub-vector.
struct CellCentroids {
    const float *coarse;
    const float *halves;
    int K;   // cells: ids outside [0, K) are invalid
    int Kh;
};

__device__ inline const float *centroid_part(const CellCentroids &cc, int c, int off, int d)
{
    if (cc.coarse) return cc.coarse + (size_t)c * d + off;
    const int dh = d >> 1;
    const int i = c / cc.Kh, j = c - i * cc.Kh;
    return off < dh ? cc.halves + (size_t)i * dh + off : cc.halves + ((size_t)cc.Kh + j) * dh + (off - dh);
}

// A wavefront takes 64 consecutive output rows, a lane each, and ENC_GROUP bytes of their codes (8 components
// of 4 bits, 4 of 8 bits, 4 of 6 bits): its lanes read neighbouring sub-vectors of their rows, the centroids
// are uniform over the wavefront (qadc_nearest.h), nothing goes through LDS, and the wavefronts of a row block
// are neighbours, so the row's lines are shared in the caches.  Before, a thread per output byte computed the
// float64 distances from a codebook in LDS, where the lanes of a wavefront met on the same banks: 2 M vectors
// of 128 dimensions, m = 16: 1029 us; residuals of 1 M vectors, m = 32: 865 us; now 277 and 208 us
// (reading the vectors at 5 TB/s takes 200 and 200 us).
// With `coarse`, row r of the output encodes the float32 residual of vector ids[r].
template <int KSUB, int DS>
__global__ __launch_bounds__(256) void pq_encode_kernel(
    const float *__restrict__ codebooks, int d, int m, const float *__restrict__ x, int64_t n,
    uint8_t *__restrict__ codes, CellCentroids cc, const int32_t *__restrict__ cells,
    const uint32_t *__restrict__ ids, int64_t n_x)
{
    constexpr int COMPS = KSUB == 16 ? 8 : 4;     // components per wavefront
    constexpr int GROUP = KSUB == 64 ? 3 : 4;     // bytes they fill
    const int dsub = DS ? DS : d / m;
    const int row = KSUB == 16 ? m / 2 : KSUB == 64 ? 3 * (m / 4) : m;
    const int groups = (m + COMPS - 1) / COMPS;
    const int64_t unit = (int64_t)blockIdx.x * (256 / WAVE) + __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const int64_t block = unit / groups;
    const int gr = (int)(unit - block * groups);
    const int64_t r = block * WAVE + (threadIdx.x & (WAVE - 1));
    if (block * WAVE >= n) return;                // uniform
    bool ok = r < n;
    const bool resid = cc.coarse || cc.halves;
    int64_t src = ids ? (ok ? (int64_t)ids[r] : 0) : (ok ? r : 0);
    int c = 0;
    if (resid) {  // an id or a cell out of range: zero bytes, no access
        if (src >= n_x) ok = false;
        if (ok) c = cells[src];
        if (c < 0 || c >= cc.K) ok = false;
    }
    // (lanes without a row read row 0 of x and cell 0; with an empty x there is nothing to read)
    if (!ok) { src = 0; c = 0; }
    const bool readable = n_x > 0;                // uniform
    // Components fetched together: a lane's loads then use up a cache line at once.  (One component at a time the
    // lines of 32 wavefronts left the L1 and the L2 between two uses: 386 us for the first of those.)
    constexpr int BATCH = DS == 0 || KSUB != 16 ? 1 : DS > 8 ? 2 : DS >= 6 ? 4 : COMPS;
    unsigned out = 0;
#pragma unroll
    for (int h0 = 0; h0 < COMPS; h0 += BATCH) {
        float xv[BATCH][DS ? DS : 1];
        const int j0 = gr * COMPS + h0;
        if (j0 >= m || !readable) break;          // uniform
        const float *xs = x + src * d + (int64_t)j0 * dsub;
        if constexpr (DS != 0) {
#pragma unroll
            for (int h = 0; h < BATCH; ++h) {
                if (j0 + h < m) {                 // uniform
#pragma unroll
                    for (int t = 0; t < DS; ++t) xv[h][t] = xs[h * DS + t];
                }
            }
            if (resid) {
#pragma unroll
                for (int h = 0; h < BATCH; ++h) {
                    if (j0 + h < m) {
                        const float *bs = centroid_part(cc, c, (j0 + h) * DS, d);
#pragma unroll
                        for (int t = 0; t < DS; ++t) xv[h][t] = xv[h][t] - bs[t];
                    }
                }
            }
        }
#pragma unroll
        for (int h = 0; h < BATCH; ++h) {
            const int j = j0 + h;
            if (j < m) {                          // uniform
                const float *bs = resid ? centroid_part(cc, c, j * dsub, d) : nullptr;
                const unsigned a = nearest_centroid<KSUB, DS>(xv[h], xs + h * dsub, bs, codebooks + (size_t)j * KSUB * dsub,
                                                              dsub, ok);
                out |= a << (KSUB == 16 ? 4 * (h0 + h) : KSUB == 64 ? 6 * (h0 + h) : 8 * (h0 + h));
            }
        }
    }
    if (r >= n) return;
    if (!ok) out = 0;
    const int64_t at = r * row + (int64_t)gr * GROUP;
    const int bytes = min(GROUP, row - gr * GROUP);
    if (GROUP == 4 && bytes == 4 && ((uintptr_t)(codes + at) & 3) == 0) {
        *reinterpret_cast<unsigned *>(codes + at) = out;
    } else {
#pragma unroll
        for (int k = 0; k < GROUP; ++k)
            if (k < bytes) codes[at + k] = (uint8_t)(out >> (8 * k));
    }
}

static int encode_launch(const char *name, const float *codebooks, int d, int m, int ksub, const float *x,
                         int64_t n, uint8_t *codes, CellCentroids cc, const int32_t *cells,
                         const uint32_t *ids, int64_t n_x, hipStream_t st)
{
    if (m < 1 || d < 1 || d % m != 0 || (ksub != 16 && ksub != 64 && ksub != 256) || (ksub == 16 && (m & 1)) ||
        (ksub == 64 && ((m & 3) || cc.coarse || cc.halves)) || n < 0)
        return fail(QADC_EINVAL, "%s: unsupported d=%d m=%d ksub=%d", name, d, m, ksub);
    if (n == 0) return QADC_OK;
    if (!codebooks || !x || !codes) return fail(QADC_EINVAL, "%s: null pointer", name);
    const int groups = (int)ceil_div(m, ksub == 16 ? 8 : 4);
    const int64_t blocks = ceil_div(ceil_div(n, WAVE) * groups, 256 / WAVE);
    if (ceil_div(n * (ksub == 16 ? m / 2 : ksub == 64 ? m / 4 : m), 256) > 0x7fffffffll || blocks > 0x7fffffffll)
        return fail(QADC_EINVAL, "%s: n too large for one call", name);
    // Sub-vectors of the usual dimensions stay in registers; with 16 centroids, whose walk is short, all up to 20 do (500 k
    // vectors of 16 x 5 components 46 us; the general form, which waits for its scalar loads, took 221).
#define QADC_ENC(K_, D_)                                                                                    \
    case D_:                                                                                                \
        hipLaunchKernelGGL((pq_encode_kernel<K_, D_>), dim3((unsigned)blocks), dim3(256), 0, st, codebooks, d, m, x, \
                           n, codes, cc, cells, ids, n_x);                                                  \
        break;
#define QADC_ENC_DS(K_, ...)                                                                                \
    switch (d / m) {                                                                                        \
    QADC_ENC(K_, 1) QADC_ENC(K_, 2) QADC_ENC(K_, 3) QADC_ENC(K_, 4) QADC_ENC(K_, 6) QADC_ENC(K_, 8) QADC_ENC(K_, 12) QADC_ENC(K_, 16) \
    __VA_ARGS__                                                                                             \
    default:                                                                                                \
        hipLaunchKernelGGL((pq_encode_kernel<K_, 0>), dim3((unsigned)blocks), dim3(256), 0, st, codebooks, d, m, x, \
                           n, codes, cc, cells, ids, n_x);                                                  \
    }
    if (ksub == 16) {
        QADC_ENC_DS(16, QADC_ENC(16, 5) QADC_ENC(16, 7) QADC_ENC(16, 9) QADC_ENC(16, 10) QADC_ENC(16, 11) QADC_ENC(16, 13)
                    QADC_ENC(16, 14) QADC_ENC(16, 15) QADC_ENC(16, 17) QADC_ENC(16, 18) QADC_ENC(16, 19) QADC_ENC(16, 20))
    } else if (ksub == 64) {
        QADC_ENC_DS(64)
    } else {
        QADC_ENC_DS(256)
    }
#undef QADC_ENC_DS
#undef QADC_ENC
    QADC_HIP_TRY(hipGetLastError());
    return QADC_OK;
}

int pq_encode(const float *codebooks, int d, int m, int ksub, const float *x, int64_t n,
              uint8_t *codes, hipStream_t st)
{
    return encode_launch("qadc_pq_encode", codebooks, d, m, ksub, x, n, codes, CellCentroids{nullptr, nullptr, 0, 0},
                         nullptr, nullptr, n, st);
}

// codes[p] = enc(x[ids[p]] - coarse[cells[ids[p]]]) for the n_list storage positions p
int ivf_encode(const float *coarse, int K, const float *codebooks, int d, int m, const float *x, int64_t n,
               const int32_t *cells, const uint32_t *ids, int64_t n_list, uint8_t *codes, hipStream_t st)
{
    if (K < 1 || n < 0) return fail(QADC_EINVAL, "qadc_ivf_encode: K=%d n=%lld", K, (long long)n);
    if (n_list > 0 && (!coarse || !cells || !ids)) return fail(QADC_EINVAL, "qadc_ivf_encode: null pointer");
    return encode_launch("qadc_ivf_encode", codebooks, d, m, 16, x, n_list, codes,
                         CellCentroids{coarse, nullptr, K, 0}, cells, ids, n, st);
}

// codes[p] = enc(x[ids[p]] - (halves[0][c / Kh], halves[1][c % Kh])), c = cells[ids[p]]
int multi_index_encode(const float *halves, int Kh, const float *codebooks, int d, int m, const float *x,
                       int64_t n, const int32_t *cells, const uint32_t *ids, int64_t n_list, uint8_t *codes,
                       hipStream_t st)
{
    if (Kh < 1 || Kh > 16384 || n < 0 || d < 2 || (d & 1))
        return fail(QADC_EINVAL, "qadc_multi_index_encode: K=%d d=%d n=%lld", Kh, d, (long long)n);
    if (n_list > 0 && (!halves || !cells || !ids)) return fail(QADC_EINVAL, "qadc_multi_index_encode: null pointer");
    return encode_launch("qadc_multi_index_encode", codebooks, d, m, 16, x, n_list, codes,
                         CellCentroids{nullptr, halves, Kh * Kh, Kh}, cells, ids, n, st);
}

}  // namespace qadc
