// Non-exhaustive search (Sections 2.2 and 2.3 of the paper) with Quick ADC on gfx950:
//   Index   squared distances of the query to the K coarse centroids, the nprobe closest cells
//   Tables  one set of m float tables per probed cell, on the residual y - centroid (Eq. (1))
//   qmax    float ADC of the first `init` codes met walking the probed lists in probe order
//           (Section 3.3), then ONE 8-bit quantizer per query shared by all its cells, so
//           that quantized sums of different cells compare
//   Scan    every code of every probed list: pair-table lookups, clamped sum (Alg. 2),
//           key = sum << 32 | storage position; R smallest keys per query; ids[position]
// Inverted lists are skewed (a few lists hold millions of codes, most a few thousand), so a
// query's lists are cut into units of at most IVF_UNIT codes; a query gets workgroups in
// proportion to its number of units, each taking a contiguous range of them.

#include <algorithm>
#include <type_traits>
#include <utility>

#include "qadc_half.h"
#include "qadc_ivf_filter.h"
#include "qadc_scan_common.h"

namespace qadc {

// f(integral_constant 0), .., f(integral_constant N - 1)
template <int... I, typename F>
__device__ __forceinline__ void static_for_each(std::integer_sequence<int, I...>, F f)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F f)
{
    static_for_each(std::make_integer_sequence<int, N>{}, f);
}

#ifndef QADC_IVF_EARLY_STAGES
// (a check at a quarter and at half of the bytes measured the same as the one check at half)
#define QADC_IVF_EARLY_STAGES(B) ((B) >= 4 ? 2 : 1)
#endif
constexpr int IVF_MAX_NPROBE = 256;
constexpr int IVF_NT = 256;      // threads of the scan workgroups
constexpr int IVF_UNIT_TILES = 8;
constexpr int IVF_WIDE_MAX_Q = 12;  // calls of up to this many queries scan with workgroups of 1024 threads

// A few queries: the tables of the probed cells stay float in memory, and every kernel that needs a
// cell's 8-bit tables applies the query's quantizer (Section 3.3) itself -- the arithmetic of
// quantize_luts_kernel, entry by entry -- which saves a pass over the tables between launches.
struct IvfQuantizer {
    const float *luts;   // [nq][nprobe][m][16]; null: the tables are quantized in memory
    const float *bias;   // [nq][m]
    const float *delta;  // [nq]
};

__device__ __forceinline__ unsigned quantize_entry(float D, float bias, float delta, unsigned nbins)
{
    const float off = fmaxf(0.0f, D - bias);
    const float t = floorf(__fdiv_rn(off, delta));
    return (t < (float)nbins) ? (unsigned)(uint8_t)t : nbins;
}

// The same from inv = 1 / delta, for delta between QUANT_INV_MIN and its inverse: off * inv is within 3 2^-24 of the rounded
// quotient, relatively, and so has the same floor unless a whole number is as near; then the division decides.  (A division
// per entry was half of the work of ivf_tables_kernel.)
constexpr float QUANT_INV_MIN = 1e-30f;
__device__ __forceinline__ unsigned quantize_entry_inv(float D, float bias, float delta, float inv, unsigned nbins)
{
    const float off = fmaxf(0.0f, D - bias);
    float t = off * inv;
    const bool near = fabsf(t - rintf(t)) < 4e-7f * t;
    if (near) t = __fdiv_rn(off, delta);
    t = floorf(t);
    return (t < (float)nbins) ? (unsigned)(uint8_t)t : nbins;
}

// entries 4 w .. 4 w + 3 of a cell's tables (inside one table: a table has 16 entries) as four bytes
__device__ __forceinline__ unsigned quantize_word(const float *cell_luts, int w, const float *bias, float delta,
                                                  unsigned nbins)
{
    const float4 v = *reinterpret_cast<const float4 *>(cell_luts + 4 * w);
    const float b = bias[w >> 2];
    return quantize_entry(v.x, b, delta, nbins) | (quantize_entry(v.y, b, delta, nbins) << 8) |
           (quantize_entry(v.z, b, delta, nbins) << 16) | (quantize_entry(v.w, b, delta, nbins) << 24);
}

// The control words of a query's scan -- the histograms of its control block and the counts of its
// report regions -- are cleared at the start of every call: calls of different shapes lay the
// workspace out differently, and what one call left as table data may lie where the next one keeps
// its counts.  Called by a whole workgroup for its query.
__device__ __forceinline__ void ivf_clear_control(char *base, size_t counts_off, int W, size_t countsA_off)
{
    unsigned *gh = reinterpret_cast<unsigned *>(base);  // ScanHeader::ghist comes first
    for (int i = threadIdx.x; i < GH_REP * 256; i += blockDim.x) gh[i] = 0;
    unsigned *counts = reinterpret_cast<unsigned *>(base + counts_off);
    for (int i = threadIdx.x; i < W; i += blockDim.x) counts[i] = 0;
    if (countsA_off && threadIdx.x == 0) *reinterpret_cast<unsigned *>(base + countsA_off) = 0;
}

// Where the kernels of the Index step clear a query's control words (calls of a few queries;
// ivf_tables_kernel does it for the others); scan_ws null: not here.
struct IvfClear {
    char *scan_ws;
    size_t ws_stride, counts_off, countsA_off;
    int W;
};

// ------------------------------------------------------------------ Index

// dist[q][c] = sum_t (y[q][t] - coarse[c][t])^2, float32, summed in increasing t with one fused
// multiply-add per component -- the same operations in the same order for a pair whatever the
// batch, so that the cells a query gets do not depend on the queries sent with it.
// A workgroup computes 16*AQ queries x 128 cells, 16 components of both at a time through LDS,
// AQ x 8 distances per thread.  Thread (tx, ty) owns queries AQ*ty.. and the cells
// 32*k + 2*tx + e, so that a wavefront's 8-byte LDS reads of the cells are contiguous.  AQ = 8
// (128 queries per workgroup).
constexpr int IVF_CT = 128;  // cells per workgroup
constexpr int IVF_CK = 16;   // components per step

// Row strides of the queries and of the distances, and what one step of blockIdx.z adds to the three arrays (the
// two halves of a multi-index; else one step).
struct IvfDistRows {
    size_t query_ld, dist_ld, coarse_z, query_z, dist_z;
};

// LISTED: only the queries list[1 .. list[0]], in their own rows.
template <int AQ, bool LISTED = false>
__global__ __launch_bounds__(256) void ivf_coarse_dist_kernel(
    const float *__restrict__ coarse, int K, int d, const float *__restrict__ queries, int nq, IvfDistRows rows,
    float *__restrict__ dist, unsigned *__restrict__ blockmin, int nblk, const unsigned *__restrict__ list)
{
    if constexpr (LISTED) {
        nq = (int)list[0];
        if ((int)blockIdx.y * 16 * AQ >= nq) return;  // uniform
    }
    auto number = [&](int q) { return LISTED ? (int)list[1 + q] : q; };
    coarse += blockIdx.z * rows.coarse_z;
    queries += blockIdx.z * rows.query_z;
    dist += blockIdx.z * rows.dist_z;
    constexpr int QT = 16 * AQ;
    __shared__ __attribute__((aligned(16))) float ys[IVF_CK][QT + 4];
    __shared__ __attribute__((aligned(16))) float cs[IVF_CK][IVF_CT + 4];
    const int tid = threadIdx.x;
    const int tx = tid & 15, ty = tid >> 4;
    const int c0 = blockIdx.x * IVF_CT;
    const int q0 = blockIdx.y * QT;
    float acc[AQ][8];
#pragma unroll
    for (int a = 0; a < AQ; ++a)
#pragma unroll
        for (int b = 0; b < 8; ++b) acc[a][b] = 0.0f;
    // the 16 components of the next step are requested while the current ones are used
    float cn[8], yn[8];
    auto fetch = [&](int t0) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int idx = tid + e * 256;
            const int row = idx >> 4, col = idx & 15;
            const int t = t0 + col;
            const int c = c0 + row;
            cn[e] = (c < K && t < d) ? coarse[(size_t)c * d + t] : 0.0f;
            yn[e] = 0.0f;
            if (row < QT) {
                const int q = q0 + row;
                if (q < nq && t < d) yn[e] = queries[(size_t)number(q) * rows.query_ld + t];
            }
        }
    };
    fetch(0);
    for (int t0 = 0; t0 < d; t0 += IVF_CK) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int idx = tid + e * 256;
            const int row = idx >> 4, col = idx & 15;
            cs[col][row] = cn[e];
            if (row < QT) ys[col][row] = yn[e];
        }
        __syncthreads();
        if (t0 + IVF_CK < d) fetch(t0 + IVF_CK);  // uniform
#pragma unroll 4
        for (int kk = 0; kk < IVF_CK; ++kk) {
            float yv[AQ], cv[8];
            if constexpr (AQ % 4 == 0) {
#pragma unroll
                for (int a = 0; a < AQ; a += 4) {
                    const float4 v = *reinterpret_cast<const float4 *>(&ys[kk][AQ * ty + a]);
                    yv[a] = v.x; yv[a + 1] = v.y; yv[a + 2] = v.z; yv[a + 3] = v.w;
                }
            } else {
#pragma unroll
                for (int a = 0; a < AQ; ++a) yv[a] = ys[kk][AQ * ty + a];
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float2 v = *reinterpret_cast<const float2 *>(&cs[kk][32 * k + 2 * tx]);
                cv[2 * k] = v.x; cv[2 * k + 1] = v.y;
            }
#pragma unroll
            for (int a = 0; a < AQ; ++a)
#pragma unroll
                for (int b = 0; b < 8; ++b) {
                    const float df = yv[a] - cv[b];
                    acc[a][b] = fmaf(df, df, acc[a][b]);
                }
        }
        __syncthreads();
    }
#pragma unroll
    for (int a = 0; a < AQ; ++a) {
        const int q = q0 + AQ * ty + a;
        const size_t at = q < nq ? number(q) : 0;  // its row
        unsigned mn = 0xffffffffu;  // smallest distance of this query over the workgroup's cells, as its image
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int c = c0 + 32 * k + 2 * tx;
            if (c < K) mn = min(mn, f2ord(acc[a][2 * k]));
            if (c + 1 < K) mn = min(mn, f2ord(acc[a][2 * k + 1]));
            if (q >= nq) continue;
            if (c + 1 < K && (rows.dist_ld & 1) == 0 && (rows.dist_z & 1) == 0) {  // the pair is 8-byte aligned
                *reinterpret_cast<float2 *>(&dist[at * rows.dist_ld + c]) = make_float2(acc[a][2 * k], acc[a][2 * k + 1]);
            } else {
                if (c < K) dist[at * rows.dist_ld + c] = acc[a][2 * k];
                if (c + 1 < K) dist[at * rows.dist_ld + c + 1] = acc[a][2 * k + 1];
            }
        }
        if (blockmin) {  // uniform: the 16 lanes tx of a query are neighbours in the wavefront
#pragma unroll
            for (int o = 1; o < 16; o <<= 1) mn = min(mn, (unsigned)__shfl_xor((int)mn, o));
            if (tx == 0 && q < nq) blockmin[at * nblk + blockIdx.x] = mn;
        }
    }
}

// The same distances for up to a few dozen queries, whose cost is one pass over the centroids: the
// workgroup's 128 centroids are requested at once (IVF_FEW_DK components of each, 64 KiB in flight per
// workgroup) and staged in LDS as they lie in memory; thread t then walks the components of cell
// t % 128, four at a time, for the queries 8 (t / 128) .. + 7 of the workgroup's 16, whose components
// every lane of the wavefront reads from the same LDS address.  Also written: the smallest distance of every
// (query, workgroup) as its order-preserving image, from which the selection kernel finds its
// threshold without reading the row.
constexpr int IVF_FEW_DK = 128;  // components staged at a time
constexpr int IVF_FEW_Q = 16;    // queries per workgroup

// acc[a] += sum over the staged components of (y_a - c)^2 for the first NQ queries of a thread: c = the
// thread's centroid row, ys = its first query's row (rows ld floats apart), four components at a time.
// (A padded component is 0 - 0: the fused multiply-add leaves the sum as it is.)
template <int NQ>
__device__ __forceinline__ void few_walk(const float *c_row, const float *ys, int ld, int dk4, float (&acc)[8])
{
    float a[NQ];
#pragma unroll
    for (int i = 0; i < NQ; ++i) a[i] = acc[i];
#pragma unroll 2
    for (int kk = 0; kk < 4 * dk4; kk += 4) {
        const float4 c = *reinterpret_cast<const float4 *>(c_row + kk);
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const float4 y = *reinterpret_cast<const float4 *>(ys + i * ld + kk);
            float df = y.x - c.x;
            a[i] = fmaf(df, df, a[i]);
            df = y.y - c.y;
            a[i] = fmaf(df, df, a[i]);
            df = y.z - c.z;
            a[i] = fmaf(df, df, a[i]);
            df = y.w - c.w;
            a[i] = fmaf(df, df, a[i]);
        }
    }
#pragma unroll
    for (int i = 0; i < NQ; ++i) acc[i] = a[i];
}

__global__ __launch_bounds__(256) void ivf_coarse_dist_few_kernel(
    const float *__restrict__ coarse, int K, int d, const float *__restrict__ queries, int nq, IvfDistRows rows,
    float *__restrict__ dist, unsigned *__restrict__ blockmin, int nblk, int vec4)
{
    coarse += blockIdx.z * rows.coarse_z;
    queries += blockIdx.z * rows.query_z;
    dist += blockIdx.z * rows.dist_z;
    constexpr int LD = IVF_FEW_DK + 4;  // rows 16-byte aligned, eight neighbouring cells on all the banks
    constexpr int QH = IVF_FEW_Q / 2;   // queries per thread
    __shared__ __attribute__((aligned(16))) float cs[IVF_CT][LD];
    __shared__ __attribute__((aligned(16))) float ys[IVF_FEW_Q][LD];
    __shared__ unsigned wmin[256 / WAVE][QH];
    const int tid = threadIdx.x;
    const int cell = tid & (IVF_CT - 1);
    const int c0 = blockIdx.x * IVF_CT;
    const int qh = QH * (tid / IVF_CT);                 // first query of this thread among the workgroup's
    const int q0 = blockIdx.y * IVF_FEW_Q + qh;         // (the same for a whole wavefront)
    const int nmine = min(QH, nq - q0);                            // its queries (may be <= 0)
    float acc[QH];
#pragma unroll
    for (int a = 0; a < QH; ++a) acc[a] = 0.0f;
    for (int t0 = 0; t0 < d; t0 += IVF_FEW_DK) {  // uniform
        const int dk = min(IVF_FEW_DK, d - t0);
        const int dk4 = (dk + 3) >> 2;  // groups of four components, the last one padded with zeros
        if (t0) __syncthreads();  // everybody is done with the previous components
        if (vec4) {  // d a multiple of four, rows 16-byte aligned
            constexpr int PER = IVF_CT * (IVF_FEW_DK / 4) / 256;  // 16 loads per thread, all in flight
            float4 v[PER];
#pragma unroll
            for (int e = 0; e < PER; ++e) {
                const int idx = tid + e * 256;
                const int row = idx / dk4, col4 = idx - row * dk4;
                v[e] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                if (row < IVF_CT && c0 + row < K)
                    v[e] = *reinterpret_cast<const float4 *>(coarse + (size_t)(c0 + row) * d + t0 + 4 * col4);
            }
            for (int idx = tid; idx < IVF_FEW_Q * dk4; idx += 256) {
                const int row = idx / dk4, col4 = idx - row * dk4;
                float4 y = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                const int q = blockIdx.y * IVF_FEW_Q + row;
                if (q < nq) y = *reinterpret_cast<const float4 *>(queries + (size_t)q * rows.query_ld + t0 + 4 * col4);
                *reinterpret_cast<float4 *>(&ys[row][4 * col4]) = y;
            }
#pragma unroll
            for (int e = 0; e < PER; ++e) {
                const int idx = tid + e * 256;
                const int row = idx / dk4, col4 = idx - row * dk4;
                if (row < IVF_CT) *reinterpret_cast<float4 *>(&cs[row][4 * col4]) = v[e];
            }
        } else {
            for (int idx = tid; idx < IVF_FEW_Q * 4 * dk4; idx += 256) {
                const int row = idx / (4 * dk4), col = idx - row * (4 * dk4);
                const int q = blockIdx.y * IVF_FEW_Q + row;
                ys[row][col] = (q < nq && col < dk) ? queries[(size_t)q * rows.query_ld + t0 + col] : 0.0f;
            }
            for (int idx = tid; idx < IVF_CT * 4 * dk4; idx += 256) {
                const int row = idx / (4 * dk4), col = idx - row * (4 * dk4);
                cs[row][col] = (c0 + row < K && col < dk) ? coarse[(size_t)(c0 + row) * d + t0 + col] : 0.0f;
            }
        }
        __syncthreads();
        if (nmine <= 0) continue;  // uniform in a wavefront: no query for it
        // the walk, compiled for every number of queries a thread can have (no test per query inside)
        switch (nmine) {
        case 1: few_walk<1>(&cs[cell][0], &ys[qh][0], IVF_FEW_DK + 4, dk4, acc); break;
        case 2: few_walk<2>(&cs[cell][0], &ys[qh][0], IVF_FEW_DK + 4, dk4, acc); break;
        case 3: few_walk<3>(&cs[cell][0], &ys[qh][0], IVF_FEW_DK + 4, dk4, acc); break;
        case 4: few_walk<4>(&cs[cell][0], &ys[qh][0], IVF_FEW_DK + 4, dk4, acc); break;
        case 5: few_walk<5>(&cs[cell][0], &ys[qh][0], IVF_FEW_DK + 4, dk4, acc); break;
        case 6: few_walk<6>(&cs[cell][0], &ys[qh][0], IVF_FEW_DK + 4, dk4, acc); break;
        case 7: few_walk<7>(&cs[cell][0], &ys[qh][0], IVF_FEW_DK + 4, dk4, acc); break;
        default: few_walk<8>(&cs[cell][0], &ys[qh][0], IVF_FEW_DK + 4, dk4, acc); break;
        }
    }
    const int c = c0 + cell;
    unsigned mn[QH];
#pragma unroll
    for (int a = 0; a < QH; ++a) {
        mn[a] = 0xffffffffu;
        if (a < nmine && c < K) {
            dist[(size_t)(q0 + a) * rows.dist_ld + c] = acc[a];
            mn[a] = f2ord(acc[a]);
        }
    }
    if (!blockmin) return;  // uniform
    // smallest image per query: inside the wavefront, then across the two wavefronts of a query
#pragma unroll
    for (int a = 0; a < QH; ++a) {
        if (a < nmine) {  // uniform in a wavefront
#pragma unroll
            for (int o = 1; o < WAVE; o <<= 1) mn[a] = min(mn[a], (unsigned)__shfl_xor((int)mn[a], o));
        }
        if (lane_id() == 0) wmin[tid / WAVE][a] = mn[a];
    }
    __syncthreads();
    if (tid < IVF_FEW_Q) {
        const int h = tid / QH, a = tid % QH;  // wavefronts 2h and 2h + 1 hold query 8h + a
        const int q = blockIdx.y * IVF_FEW_Q + tid;
        if (q < nq) blockmin[(size_t)q * nblk + blockIdx.x] = min(wmin[2 * h][a], wmin[2 * h + 1][a]);
    }
}

// The distances of nq queries to K centroids (`parts` times, see IvfDistRows).  The tiled kernel reads a centroid
// once for 128 queries; where its workgroups would leave most of the GPU idle (a few hundred cells), or for up
// to 32 queries, the kernel for 16 queries is the faster one: 150 queries x 256 cells 12 against 44 us.
void ivf_distances(const float *coarse, int K, int d, const float *queries, int nq, IvfDistRows rows, int parts,
                   float *dist, unsigned *bmin, hipStream_t st)
{
    const int nblk = (int)ceil_div(K, IVF_CT);
    const int64_t tiles = (int64_t)nblk * ceil_div(nq, 128) * parts;
    if (nq > 32 && tiles >= 256) {
        dim3 grid((unsigned)nblk, (unsigned)ceil_div(nq, 128), (unsigned)parts);
        launch(QADC_PROF_IVF_INDEX, ivf_coarse_dist_kernel<8>, grid, dim3(256), 0, st, coarse, K, d, queries, nq, rows,
               dist, bmin, nblk, (const unsigned *)nullptr);
    } else {
        const int vec4 = (d % 4 == 0 && rows.query_ld % 4 == 0 && rows.query_z % 4 == 0 && rows.coarse_z % 4 == 0 &&
                          ((uintptr_t)coarse & 15) == 0 && ((uintptr_t)queries & 15) == 0) ? 1 : 0;
        dim3 grid((unsigned)nblk, (unsigned)ceil_div(nq, IVF_FEW_Q), (unsigned)parts);
        launch(QADC_PROF_IVF_INDEX, ivf_coarse_dist_few_kernel, grid, dim3(256), 0, st, coarse, K, d, queries, nq, rows,
               dist, bmin, nblk, vec4);
    }
}

// The 2 K half distances of nq queries: hd[(q * 2 + h)][i] to half-centroid i of half h.
void multi_half_distances(const float *halves, int K, int dh, const float *queries, int nq, float *hd, hipStream_t st)
{
    const IvfDistRows rows = {(size_t)(2 * dh), (size_t)(2 * K), (size_t)K * dh, (size_t)dh, (size_t)K};
    ivf_distances(halves, K, dh, queries, nq, rows, 2, hd, nullptr, st);
}

// probes[q][0..nprobe) = the nprobe closest cells, closest first, ties to the lowest cell id.
// Keys are order(dist) << 32 | cell (unique).  Thread t looks at cells t, t + NT, ...  The
// need-th smallest of the threads' minima, T, bounds the need-th smallest key of the whole
// row from above (need threads each hold a key <= T), and only those need threads can hold
// keys <= T: at most need * ceil(K / NT) candidates, normally about `need` of them.  A second
// pass over the row gathers the candidates in LDS, where the exact selection runs.  A
// candidate list that does not fit takes the radix select over the whole row instead.
// With `blockmin` (the smallest distance of every run of IVF_CT cells, at least `need` runs): T = the
// need-th smallest of those minima, by the same argument, and only the runs whose minimum is <= T are
// read at all -- the row is not walked twice by one workgroup.
constexpr int IVF_SEL_NT = 1024;
constexpr int IVF_SEL_CAP = 4096;
constexpr int IVF_SEL_MAXBLK = 4096;  // runs of cells whose minima fit in LDS

// The end of a selection, by a workgroup of IVF_SEL_NT threads after a barrier: of the cnt candidates (keys order(dist) <<
// 32 | cell) in LDS -- of the whole row of distances where there are more than fit -- the `need` smallest in order, and
// unused slots behind them.
__device__ __forceinline__ void probes_of_candidates(const float *dq, int K, int nprobe, unsigned need, uint64_t *cand,
                                                     unsigned &cnt, SelectScratch &sc, int32_t *__restrict__ probes)
{
    constexpr int NT = IVF_SEL_NT;
    const int tid = threadIdx.x;
    const unsigned ncand = cnt;
    const bool in_lds = ncand <= (unsigned)IVF_SEL_CAP;
    __syncthreads();

    auto each_row = [&](auto f) {
        for (int c = tid; c < K; c += NT) f(((uint64_t)f2ord(dq[c]) << 32) | (uint64_t)(unsigned)c);
    };
    if (ncand <= (unsigned)NT) {
        // a thread per candidate: its rank among all of them is its place among the probes
        if ((unsigned)tid < ncand) {
            const uint64_t k = cand[tid];
            unsigned rank = 0;
            for (unsigned j = 0; j < ncand; ++j) rank += (cand[j] < k) ? 1u : 0u;
            if (rank < need) probes[rank] = (int32_t)(unsigned)k;
        }
        for (unsigned i = need + tid; i < (unsigned)nprobe; i += NT) probes[i] = -1;
        return;  // uniform
    }
    uint64_t kth;
    if (in_lds) kth = block_radix_select<uint64_t, 8>(cand, ncand, need, &sc);
    else kth = block_radix_select_each<uint64_t, 8>(each_row, need, &sc);
    // the winners (exactly `need`: keys are unique), ordered by rank
    __shared__ uint64_t sel[IVF_MAX_NPROBE];
    if (tid == 0) cnt = 0;
    __syncthreads();
    if (in_lds) {
        for (unsigned i = tid; i < ncand; i += NT)
            if (cand[i] <= kth) sel[atomicAdd(&cnt, 1u)] = cand[i];
    } else {
        each_row([&](uint64_t k) {
            if (k <= kth) sel[atomicAdd(&cnt, 1u)] = k;
        });
    }
    __syncthreads();
    for (unsigned i = tid; i < (unsigned)nprobe; i += NT) {
        if (i >= need) {
            probes[i] = -1;
        } else {
            const uint64_t k = sel[i];
            unsigned rank = 0;
            for (unsigned j = 0; j < need; ++j) rank += (sel[j] < k) ? 1u : 0u;
            probes[rank] = (int32_t)(unsigned)k;
        }
    }
}


// LISTED: as in ivf_coarse_dist_kernel.
template <bool LISTED>
__global__ __launch_bounds__(IVF_SEL_NT) void ivf_select_probes_kernel(
    const float *__restrict__ dist, int K, int nprobe, int32_t *__restrict__ probes,
    const unsigned *__restrict__ blockmin, int nblk, IvfClear clr, const unsigned *__restrict__ list)
{
    constexpr int NT = IVF_SEL_NT;
    if (LISTED && blockIdx.x >= list[0]) return;  // uniform
    if (clr.scan_ws) {  // uniform
        ivf_clear_control(clr.scan_ws + (size_t)blockIdx.x * clr.ws_stride, clr.counts_off, clr.W, clr.countsA_off);
    }
    __shared__ SelectScratch sc;
    __shared__ uint64_t cand[IVF_SEL_CAP];  // thread minima first, then the candidates
    __shared__ unsigned cnt;
    const int tid = threadIdx.x;
    const int q = LISTED ? (int)list[1 + blockIdx.x] : (int)blockIdx.x;
    const float *dq = dist + (size_t)q * K;
    const unsigned need = (unsigned)min(nprobe, K);

    if (blockmin) {  // uniform
        __shared__ unsigned bm[IVF_SEL_MAXBLK];
        __shared__ unsigned hits[IVF_SEL_MAXBLK];
        __shared__ unsigned nhit_s;
        for (int b = tid; b < nblk; b += NT) bm[b] = blockmin[(size_t)q * nblk + b];
        if (tid == 0) { cnt = 0; nhit_s = 0; }
        __syncthreads();
        // the three leading bytes of the need-th smallest minimum, everything below them set
        unsigned Tm = block_radix_select_each<unsigned, 3>(
            [&](auto f) {
                for (int b = tid; b < nblk; b += NT) f(bm[b] >> 8);
            },
            need, &sc);
        Tm = (Tm << 8) | 0xffu;
        for (int b = tid; b < nblk; b += NT)
            if (bm[b] <= Tm) hits[atomicAdd(&nhit_s, 1u)] = (unsigned)b;
        __syncthreads();
        const unsigned ncell = nhit_s * (unsigned)IVF_CT;
        for (unsigned i0 = tid; i0 < ncell; i0 += 4 * NT) {
            float v[4];
            int c[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const unsigned i = i0 + u * NT;
                c[u] = i < ncell ? (int)(hits[i / IVF_CT] * IVF_CT + i % IVF_CT) : K;
                v[u] = c[u] < K ? dq[c[u]] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const unsigned o = f2ord(v[u]);
                if (c[u] < K && o <= Tm) {
                    const unsigned slot = atomicAdd(&cnt, 1u);
                    if (slot < (unsigned)IVF_SEL_CAP) cand[slot] = ((uint64_t)o << 32) | (uint64_t)(unsigned)c[u];
                }
            }
        }
    } else {
    // this thread's smallest key: smallest value, lowest cell among equals (cells grow with c)
    // (eight loads in flight per thread: the row is read at memory speed, not one latency per cell)
    uint64_t mine = ~0ull;
    for (int c0 = tid; c0 < K; c0 += 8 * NT) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int c = c0 + u * NT;
            v[u] = c < K ? dq[c] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int c = c0 + u * NT;
            if (c < K) mine = min(mine, ((uint64_t)f2ord(v[u]) << 32) | (uint64_t)(unsigned)c);
        }
    }
    const int nmin = min(K, NT);  // threads that hold at least one key
    if (tid < nmin) cand[tid] = mine;
    if (tid == 0) cnt = 0;
    __syncthreads();
    // Any T at or above the need-th smallest minimum will do: the three leading bytes of the
    // distance decide it (three histogram passes instead of eight), everything below is set.
    uint64_t T = block_radix_select_each<uint64_t, 3>(
        [&](auto f) {
            for (int i = tid; i < nmin; i += NT) f(cand[i] >> 40);
        },
        need, &sc);
    T = (T << 40) | 0xffffffffffull;
    __syncthreads();  // everybody has T; the minima may be overwritten
    // second pass over the row, by every thread as the first (only a thread whose minimum is <= T
    // finds anything, but a few threads walking their cells alone would pay a latency per cell)
    for (int c0 = tid; c0 < K; c0 += 8 * NT) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int c = c0 + u * NT;
            v[u] = c < K ? dq[c] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int c = c0 + u * NT;
            const uint64_t k = ((uint64_t)f2ord(v[u]) << 32) | (uint64_t)(unsigned)c;
            if (c < K && k <= T) {
                const unsigned slot = atomicAdd(&cnt, 1u);
                if (slot < (unsigned)IVF_SEL_CAP) cand[slot] = k;
            }
        }
    }
    }
    __syncthreads();
    probes_of_candidates(dq, K, nprobe, need, cand, cnt, sc, probes + (size_t)q * nprobe);
}

// The same from the bounds of qadc_ivf_filter.hip, one per group of four cells, in the query's row of `dist`: any T that `need`
// groups do not exceed bounds the need-th smallest score (as above, the need-th smallest of the threads' minima), and with
// the rounding of the scores and of float32 distances (components + 4 roundings of 2^-24) the scores of all cells among the
// `need` closest.  The cells of those groups -- some 70 groups for 64 probes -- are measured by the definition
// (ivf_coarse_dist_kernel's operations in its order), a thread per cell.  A query that this cannot serve (beyond the range of
// the factors, too many groups as close, a NaN anywhere) goes to `rest` (their number, then the queries in any order), for the
// float32 distances to all cells (2000 queries, 16,334 of 16,384 centroids in one place: 1310 us; measured against all
// cells by its own workgroup instead, 2670: the centroids from the caches once per query).
constexpr int IVF_SEL_GROUPS = IVF_SEL_CAP / 4;

__global__ __launch_bounds__(IVF_SEL_NT) void ivf_select_filtered_kernel(
    const float *__restrict__ coarse, int K, int d, const float *__restrict__ queries, float *__restrict__ dist,
    const float2 *__restrict__ qstat, int components, int nprobe, int32_t *__restrict__ probes, int vec4,
    unsigned *__restrict__ rest)
{
    constexpr int NT = IVF_SEL_NT;
    __shared__ SelectScratch sc;
    __shared__ uint64_t cand[IVF_SEL_CAP];
    __shared__ unsigned small_s[NT];
    __shared__ unsigned groups[IVF_SEL_GROUPS];
    __shared__ __attribute__((aligned(16))) float ys[256];
    __shared__ unsigned cnt, ngroup;
    const int tid = threadIdx.x;
    const int q = blockIdx.x;
    const unsigned need = (unsigned)min(nprobe, K);
    const int tiles = (K + 31) / 32;
    if (tid < d) ys[tid] = queries[(size_t)q * d + tid];
    const float2 stat = qstat[q];
    const unsigned *row = reinterpret_cast<const unsigned *>(ivf_filter_row(dist, K, (size_t)q));  // two bounds a word
    auto order = [](unsigned b) { return (b & 0x8000u) ? ~b & 0xffffu : b | 0x8000u; };
    auto each_pair = [&](auto f) {  // f(first group, its key, the next one's key)
        for (int i0 = tid; i0 < 4 * tiles; i0 += 8 * NT) {
            unsigned w[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) w[u] = i0 + u * NT < 4 * tiles ? row[i0 + u * NT] : 0x7f807f80u;
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (i0 + u * NT < 4 * tiles) f(2 * (i0 + u * NT), order(w[u] & 0xffffu), order(w[u] >> 16));
        }
    };
    unsigned mine = 0xffffu;
    each_pair([&](int, unsigned k0, unsigned k1) { mine = min(mine, min(k0, k1)); });
    const int nmin = min(NT, 4 * tiles);  // (at least `need`: the host sees to it)
    small_s[tid] = mine;
    if (tid == 0) { cnt = 0; ngroup = 0; }
    const bool nan = __syncthreads_or(mine <= order(0xff80u));  // minus infinity: a centroid with a NaN
    const unsigned T = block_radix_select_each<unsigned, 2>(
        [&](auto f) {
            if (tid < nmin) f(small_s[tid]);
        },
        need, &sc);
    auto value = [](unsigned o) { return __uint_as_float(((o & 0x8000u) ? o & 0x7fffu : ~o & 0xffffu) << 16); };
    const float up = value(T + 1u);  // no bound that was rounded to T is beyond the next bfloat16
    const float xn = stat.x, tiny = HALF_TINY * (float)components;
    const float xerr = __builtin_fmaf(half_eps(components), xn, __builtin_fmaf(HALF_CONV, stat.y, tiny));
    const float far = 1.05f * (__builtin_sqrtf(xn) + __builtin_sqrtf(fmaxf(up + xerr + 2.0f * tiny, 0.0f)));
    const float cerr = __builtin_fmaf(1.01f * half_eps_c(components), far * far, tiny);
    const float reach = up + xerr + 2.002f * cerr;  // squared distance (scaled) of the need-th closest cell, at most
    const float thr = __builtin_fmaf(reach, 2e-7f * (float)(components + 4), reach) + 1.001f * xerr;
    // (comparisons that a NaN fails)
    const bool sure = !nan && T < 0xff7fu && xn < HALF_NEAR && up - xn < HALF_FAR && thr < 4.0f * HALF_FAR;  // uniform
    if (sure) {
        const __bf16 rounded = (__bf16)thr;
        const unsigned last = order(__builtin_bit_cast(uint16_t, rounded));
        each_pair([&](int g, unsigned k0, unsigned k1) {
            if (min(k0, k1) <= last) {
                if (k0 <= last) {
                    const unsigned slot = atomicAdd(&ngroup, 1u);
                    if (slot < (unsigned)IVF_SEL_GROUPS) groups[slot] = (unsigned)g;
                }
                if (k1 <= last) {
                    const unsigned slot = atomicAdd(&ngroup, 1u);
                    if (slot < (unsigned)IVF_SEL_GROUPS) groups[slot] = (unsigned)g + 1u;
                }
            }
        });
    }
    __syncthreads();
    const unsigned ng = ngroup;
    if (!sure || ng > (unsigned)IVF_SEL_GROUPS) {  // uniform
        if (tid == 0) rest[1 + atomicAdd(rest, 1u)] = (unsigned)q;
        return;
    }
    auto measure = [&](int c) {
        const float *cr = coarse + (size_t)c * d;
        float acc = 0.0f;
        if (vec4) {  // uniform
#pragma unroll 8
            for (int t = 0; t < d; t += 4) {
                const float4 v = *reinterpret_cast<const float4 *>(cr + t);
                const float4 y = *reinterpret_cast<const float4 *>(&ys[t]);
                float df = y.x - v.x;
                acc = fmaf(df, df, acc);
                df = y.y - v.y;
                acc = fmaf(df, df, acc);
                df = y.z - v.z;
                acc = fmaf(df, df, acc);
                df = y.w - v.w;
                acc = fmaf(df, df, acc);
            }
        } else {
#pragma unroll 8
            for (int t = 0; t < d; ++t) {
                const float df = ys[t] - cr[t];
                acc = fmaf(df, df, acc);
            }
        }
        return acc;
    };
    float *dq = dist + (size_t)q * K;
    for (unsigned i = tid; i < 4u * ng; i += NT) {
        const int c = (int)(ivf_filter_first_cell(groups[i >> 2]) + (i & 3u));
        if (c < K) cand[atomicAdd(&cnt, 1u)] = ((uint64_t)f2ord(measure(c)) << 32) | (uint64_t)(unsigned)c;
    }
    __syncthreads();
    probes_of_candidates(dq, K, nprobe, need, cand, cnt, sc, probes + (size_t)q * nprobe);
}

// rows of `dist` [rows][K] -> out[rows][count]: the count smallest of each row, smallest first
// (for the multi-index's half distances)
void ivf_select_smallest(const float *dist, int rows, int K, int count, int32_t *out, hipStream_t st)
{
    launch(QADC_PROF_IVF_INDEX, ivf_select_probes_kernel<false>, dim3((unsigned)rows), dim3(IVF_SEL_NT), 0, st, dist, K,
           count, out, (const unsigned *)nullptr, 0, IvfClear{nullptr, 0, 0, 0, 0}, (const unsigned *)nullptr);
}

// ----------------------------------------------------------------- Tables

// Float tables of the probed cells for ivf_tables_kernel<0>: luts[q][p][j][i] = || (y_q - centroid_p)^j - C^j[i] ||^2, float64
// inside, one rounding to float32; +inf for unused probe slots (cell id < 0).
// A workgroup takes CELLS of a query's cells and reads the codebooks once for them, a thread per entry; the cells' residuals
// are in LDS as float64, tables a component apart from each other against bank conflicts (CELLS = 0: no room for them, d beyond
// 8000 or so; taken from memory for every entry).  Bound by the reads of the codebooks, rows d / m floats apart.
// us for the tables of 64 probed cells, as they are here / an entry by the query's one workgroup, from memory, twice: 40 queries
// d = 960, m = 32 47 / 902, 500 137 / 3413, d = 96, m = 32 32 / 112, 40 queries d = 200, m = 8 21 / 142.
template <int CELLS>
__global__ __launch_bounds__(256) void ivf_float_tables_kernel(
    const float *__restrict__ codebooks, int d, int m, const float *__restrict__ queries,
    const float *__restrict__ coarse, const float *__restrict__ halves, const uint32_t *__restrict__ cell_ids,
    int Kh, const int32_t *__restrict__ probes, int nprobe, float *__restrict__ luts)
{
    extern __shared__ double res[];  // [CELLS][m][dsub + 1]
    constexpr int N = CELLS ? CELLS : 1;
    const int q = blockIdx.y, p0 = blockIdx.x * N;
    const int dsub = d / m, dh = d >> 1, pitch = dsub + 1;
    const int entries = m * 16;
    const float *yq = queries + (size_t)q * d;
    const float *row[N][2];  // the centroid's components of the first and of the second half (null: no cell)
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const int cell = p0 + k < nprobe ? probes[(size_t)q * nprobe + p0 + k] : -1;
        row[k][0] = row[k][1] = nullptr;
        if (cell >= 0) {
            if (coarse) {
                row[k][0] = row[k][1] = coarse + (size_t)cell * d;
            } else {  // list `cell` of a multi-index: the centroid is a pair of half-centroids
                const unsigned id = cell_ids[cell];
                row[k][0] = halves + (size_t)(id / (unsigned)Kh) * dh;
                row[k][1] = halves + ((size_t)Kh + id % (unsigned)Kh) * dh - dh;
            }
        }
    }
    auto residual = [&](int k, int t) {
        const float *r = coarse || t < dh ? row[k][0] : row[k][1];
        return (double)yq[t] - (r ? (double)r[t] : 0.0);
    };
    if constexpr (CELLS > 0) {
        for (int t = threadIdx.x; t < d; t += 256) {
            const int at = t + t / dsub;
#pragma unroll
            for (int k = 0; k < N; ++k) res[k * m * pitch + at] = residual(k, t);
        }
        __syncthreads();
    }
    for (int e = threadIdx.x; e < entries; e += 256) {
        const float *c = codebooks + (size_t)e * dsub;
        const int j = e >> 4;
        double acc[N];
#pragma unroll
        for (int k = 0; k < N; ++k) acc[k] = 0.0;
        auto add = [&](int t, float cv) {
#pragma unroll
            for (int k = 0; k < N; ++k) {
                const double df = (CELLS > 0 ? res[k * m * pitch + j * pitch + t] : residual(k, j * dsub + t)) - (double)cv;
                acc[k] += df * df;
            }
        };
        int t0 = 0;
        for (; t0 + 8 <= dsub; t0 += 8) {
            float cv[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) cv[t] = c[t0 + t];
#pragma unroll
            for (int t = 0; t < 8; ++t) add(t0 + t, cv[t]);
        }
        for (; t0 < dsub; ++t0) add(t0, c[t0]);
#pragma unroll
        for (int k = 0; k < N; ++k)
            if (p0 + k < nprobe)
                luts[((size_t)q * nprobe + p0 + k) * entries + e] = row[k][0] ? (float)acc[k] : __builtin_inff();
    }
}

// Batches: Tables, the qmax walk and the quantizer by one workgroup per query, a thread per table entry and, where the
// tables are smaller than the workgroup, per one of several probed cells at a time.  Entry (j, i) of cell p is
// || (y_q - centroid_p)^j - C^j[i] ||^2, float64 inside, one rounding to float32 (as the exhaustive tables kernel); unused
// probe slots (cell id < 0) have +inf tables: nothing of them is ever scanned.
//   1. qmax = min(R, n_walk)-th smallest float ADC distance (Eq. (2), float32, increasing j) of the first n_walk =
//      min(init, codes in the probed lists) codes met walking the lists in probe order, each code with the tables of its
//      own cell; 0 when the lists are empty.  The tables of the lists walked pass through LDS.
//   2. bias_j = smallest entry of table j over all probed cells.
//   3. the entries again, quantized (the arithmetic of quantize_luts_kernel).
// Bound by its float64 instructions and, below some 500 queries, by the chain of steps of one workgroup.  A thread's first KEEP
// entries stay in registers between steps 2 and 3, those beyond are computed twice (128 registers; the forms of 4 and 8
// components spill 6 of them, that of 16 16): as three kernels, the float tables of 4096 queries x 64 cells were 537 MB written by
// one, gathered from by the second and read by the third, 560 us (m = 32, d = 128) against 335 now; 512 queries 82 against 49,
// 150 queries x 24 cells (m = 16) 25 against 12.  (Every entry computed twice instead, with no registers held: 64 us for the
// 512.  Every lane converting its own residuals: 51.)
// Other lengths (DSUB = 0), and calls for which that chain is too long (ivf_tables_form): the entries come from memory, where
// ivf_float_tables_kernel has left them, and are read once.
constexpr int IVF_WALK = 4;  // lists walked at a time, per table set that the workgroup's threads are
template <int DSUB>  // d / m; 0: any, the entries from `luts`
__global__ __launch_bounds__(1024) void ivf_tables_kernel(
    const float *__restrict__ codebooks, int d, int m, const float *__restrict__ queries,
    const float *__restrict__ coarse, const float *__restrict__ halves, const uint32_t *__restrict__ cell_ids,
    int Kh, const int32_t *__restrict__ probes, int nprobe, const float *__restrict__ luts, const int64_t *__restrict__ list_off,
    const uint8_t *__restrict__ codes, int64_t n_total, int init, int R, int nbins, int qmin_mode, long long unit,
    unsigned *__restrict__ qunits, uint8_t *__restrict__ qluts, char *__restrict__ ws, size_t ws_stride,
    size_t counts_off, int W, size_t countsA_off, unsigned *__restrict__ pair_cnt, int K)
{
    ivf_clear_control(ws + (size_t)blockIdx.x * ws_stride, counts_off, W, countsA_off);
    if (pair_cnt)  // the shared-list scan's counts of pairs per cell, taken by the kernel after this one
        for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < K; i += (int64_t)gridDim.x * blockDim.x) pair_cnt[i] = 0;
    __shared__ unsigned cand[QADC_MAX_INIT];
    __shared__ float lut_s[IVF_WALK][1024];
    __shared__ unsigned units_s;
    __shared__ long long start[IVF_MAX_NPROBE + 1];  // codes before probe p in the walk
    __shared__ long long lo[IVF_MAX_NPROBE];
    __shared__ int row0[IVF_MAX_NPROBE], row1[IVF_MAX_NPROBE];  // the centroid, or the two half-centroids, of probe p; -1
    __shared__ unsigned bias_ord[64];
    __shared__ float bias[64];
    __shared__ float delta_s;
    __shared__ SelectScratch sc;
    __shared__ unsigned long long wsum[1024 / WAVE];
    const int q = blockIdx.x;
    const int tid = threadIdx.x, NT = blockDim.x;
    const int B = m / 2;
    const int entries = m * 16;              // a power of two that divides NT
    const int e = tid & (entries - 1);       // entry: table j = e / 16, centroid e % 16
    const int sub = tid / entries, subs = NT / entries;
    const int j = e >> 4;
    const int dsub = DSUB ? DSUB : d / m;
    const int t0 = j * dsub;
    // list lengths one thread per probe, exclusive prefix sum
    unsigned long long len = 0;
    if (tid == 0) units_s = 0;
    if (tid < 64) bias_ord[tid] = 0xffffffffu;
    __syncthreads();
    if (tid < nprobe) {
        const int cell = probes[(size_t)q * nprobe + tid];
        long long l = 0, h = 0;
        int r0 = -1, r1 = -1;
        if (cell >= 0) {
            l = list_off[cell];
            h = list_off[cell + 1];
            r0 = r1 = cell;
            if (!coarse) {  // list `cell` of a multi-index: the centroid is a pair of half-centroids
                const unsigned id = cell_ids[cell];
                r0 = (int)(id / (unsigned)Kh);
                r1 = (int)(id % (unsigned)Kh);
            }
        }
        if (l < 0 || h > n_total || h < l) l = h = 0;  // offsets that are not a list: nothing is read
        lo[tid] = l;
        row0[tid] = r0;
        row1[tid] = r1;
        len = (unsigned long long)(h - l);
        // units the scan kernel cuts this list into (the same expression as there)
        if (h > l) atomicAdd(&units_s, (unsigned)((h - l / 16 * 16 + unit - 1) / unit));
    }
    {
        const int l = lane_id();
        unsigned long long inc = len;
#pragma unroll
        for (int dd = 1; dd < WAVE; dd <<= 1) {
            const unsigned long long up = __shfl_up(inc, dd);
            if (l >= dd) inc += up;
        }
        if (l == WAVE - 1) wsum[tid / WAVE] = inc;
        __syncthreads();
        unsigned long long before = 0;
        for (int wv = 0; wv < tid / WAVE; ++wv) before += wsum[wv];
        if (tid < nprobe) start[tid] = (long long)(before + inc - len);
        if (tid == nprobe - 1) start[nprobe] = (long long)(before + inc);
    }
    __syncthreads();
    if (tid == 0) qunits[q] = units_s;

    // this thread's centroid and sub-vector of the query, and where its sub-vector of a cell's centroid lies
    constexpr int REGS = DSUB ? DSUB : 1;
    double c[REGS];
    if constexpr (DSUB > 0) {
#pragma unroll
        for (int t = 0; t < DSUB; ++t) c[t] = (double)codebooks[(size_t)e * DSUB + t];
    }
    const int dh = d >> 1;
    const bool first = coarse || t0 < dh;  // (a sub-vector lies inside one half)
    const float *base = coarse ? coarse + t0 : t0 < dh ? halves + t0 : halves + (size_t)Kh * dh + (t0 - dh);
    const size_t ld = coarse ? (size_t)d : (size_t)dh;
    auto row_of = [&](int p) { return first ? row0[p] : row1[p]; };
    auto entry = [&](int p) {
        if constexpr (DSUB == 0) return luts[((size_t)q * nprobe + p) * entries + e];
        return 0.0f;
    };
    // The same for SIDE probes at a time: the 16 lanes of a table need the same residuals y - centroid, so lane k % 16 takes
    // component k % DSUB of probe k / DSUB, and the others get it from there.  (Every lane for itself, conversions and
    // differences were the larger part of the kernel: 16 conversions to float64 per four entries instead of one.)
    constexpr int SIDE = DSUB > 0 ? 16 / DSUB : 1;
    constexpr int AHEAD = DSUB == 2 ? 2 : 4;  // groups of SIDE probes whose centroids are requested together
    const int own = DSUB > 0 ? min((e & 15) / REGS, SIDE - 1) : 0, own_t = DSUB > 0 ? (e & 15) % REGS : 0;
    const double own_y = DSUB > 0 ? (double)queries[(size_t)q * d + t0 + own_t] : 0.0;
    auto residuals = [&](int p) {  // of probes p, p + subs, .. (the last probe's beyond it): this lane's
        const float *r = base + (size_t)max(row_of(min(p + own * subs, nprobe - 1)), 0) * ld;
        return own_y - (double)r[own_t];
    };
    auto entries_of = [&](int p, double res, float (&v)[SIDE]) {
        const int lo32 = (int)__builtin_bit_cast(unsigned long long, res), hi32 = (int)(__builtin_bit_cast(unsigned long long, res) >> 32);
        auto from = [&](auto lane) {
            constexpr int bcast = 0x150 + decltype(lane)::value;  // to the 16 lanes from this one of theirs
            const unsigned l = (unsigned)__builtin_amdgcn_mov_dpp(lo32, bcast, 0xf, 0xf, true);
            const unsigned h = (unsigned)__builtin_amdgcn_mov_dpp(hi32, bcast, 0xf, 0xf, true);
            return __builtin_bit_cast(double, (unsigned long long)l | ((unsigned long long)h << 32));
        };
        static_for<SIDE>([&](auto a) {
            double acc = 0.0;
            static_for<REGS>([&](auto t) {
                const double df = from(std::integral_constant<int, decltype(a)::value * REGS + decltype(t)::value>{}) - c[decltype(t)::value];
                acc += df * df;
            });
            v[decltype(a)::value] = row_of(min(p + decltype(a)::value * subs, nprobe - 1)) < 0 ? __builtin_inff() : (float)acc;
        });
    };
    // f(p, entry) for this thread's probes from p0 on
    auto each_probe = [&](int p0, auto f) {
        constexpr int STEP = DSUB > 0 ? SIDE : 8;
        for (int p = p0 + sub; p < nprobe; p += STEP * subs) {  // uniform in a wavefront
            float v[STEP];
            if constexpr (DSUB > 0) {
                entries_of(p, residuals(p), v);
            } else {
#pragma unroll
                for (int a = 0; a < STEP; ++a) v[a] = entry(min(p + a * subs, nprobe - 1));
            }
#pragma unroll
            for (int a = 0; a < STEP; ++a)
                if (p + a * subs < nprobe) f(p + a * subs, v[a]);
        }
    };

    const int n_walk = (int)min((long long)init, start[nprobe]);
    const int walked = __syncthreads_count(tid < nprobe && start[min(tid, nprobe)] < n_walk);  // lists with a code of the walk before their end
    unsigned least = 0xffffffffu;  // smallest value of this entry, as its order-preserving image
    for (int p0 = 0; p0 < walked; p0 += IVF_WALK * subs) {  // uniform
        if constexpr (DSUB == 0) {
#pragma unroll
            for (int a = 0; a < IVF_WALK; ++a) lut_s[a][tid] = entry(min(p0 + sub + a * subs, nprobe - 1));
        } else {
            constexpr int AT_ONCE = SIDE < IVF_WALK ? SIDE : IVF_WALK;
#pragma unroll
            for (int a0 = 0; a0 < IVF_WALK; a0 += AT_ONCE) {
                if (p0 + a0 * subs >= walked) break;  // uniform
                float v[SIDE];
                entries_of(p0 + sub + a0 * subs, residuals(p0 + sub + a0 * subs), v);
#pragma unroll
                for (int a = 0; a < AT_ONCE; ++a) lut_s[a0 + a][tid] = v[a];
            }
        }
        __syncthreads();
        const int s1 = (int)min(start[min(p0 + IVF_WALK * subs, walked)], (long long)n_walk);
        for (int i = (int)start[p0] + tid; i < s1; i += NT) {
            int p = p0;
            while (start[p + 1] <= i) ++p;
            // the code as 32-bit words (B is a multiple of 4, up to 32), all requested at once: the sum keeps the order of j
            const unsigned *cw = reinterpret_cast<const unsigned *>(codes + (size_t)(lo[p] + (i - start[p])) * B);
            const float *lut = &lut_s[0][0] + (p - p0) / subs * 1024 + (p - p0) % subs * entries;
            unsigned w[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) w[k] = 4 * k < B ? cw[k] : 0u;  // (uniform)
            float acc = 0.0f;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                if (4 * k < B) {  // uniform
                    float ent[8];
#pragma unroll
                    for (int b = 0; b < 4; ++b) {
                        const unsigned comps = (w[k] >> (8 * b)) & 0xffu;
                        const int jb = 4 * k + b;
                        ent[2 * b] = lut[(2 * jb) * 16 + (comps & 15u)];
                        ent[2 * b + 1] = lut[(2 * jb + 1) * 16 + (comps >> 4)];
                    }
#pragma unroll
                    for (int b = 0; b < 8; ++b) acc = acc + ent[b];
                }
            }
            cand[i] = f2ord(acc);
        }
        __syncthreads();
    }
    // the entries of the first KEEP probes of the thread stay in registers for step 3, those beyond are computed twice
    constexpr int KEEP = DSUB <= 4 ? 64 : 32, BLOCK = DSUB > 0 ? AHEAD * SIDE : 8;
    static_assert(KEEP % BLOCK == 0, "whole blocks");
    float kept[KEEP ? KEEP : 1];
#pragma unroll
    for (int k = 0; k < KEEP; k += BLOCK) {
        if (k * subs < nprobe) {  // uniform
            // (the last probe again where there is none)
            if constexpr (DSUB == 0) {
#pragma unroll
                for (int a = 0; a < BLOCK; ++a) kept[k + a] = entry(min(sub + (k + a) * subs, nprobe - 1));
#pragma unroll
                for (int a = 0; a < BLOCK; ++a) least = min(least, f2ord(kept[k + a]));
            } else {
                double res[AHEAD];
#pragma unroll
                for (int a = 0; a < AHEAD; ++a) res[a] = residuals(sub + (k + a * SIDE) * subs);
#pragma unroll
                for (int a = 0; a < AHEAD; ++a) {
                    float v[SIDE];
                    entries_of(sub + (k + a * SIDE) * subs, res[a], v);
#pragma unroll
                    for (int i = 0; i < SIDE; ++i) {
                        kept[k + a * SIDE + i] = v[i];
                        least = min(least, f2ord(v[i]));
                    }
                }
            }
        }
    }
    each_probe(KEEP * subs, [&](int, float v) { least = min(least, f2ord(v)); });
#pragma unroll
    for (int w = 8; w >= 1; w >>= 1) least = min(least, (unsigned)__shfl_xor((int)least, w));
    if ((e & 15) == 0) atomicMin(&bias_ord[j], least);
    float qmax = 0.0f;
    if (n_walk > 0)  // uniform
        qmax = ord2f(block_radix_select<unsigned, 4>(cand, (unsigned)n_walk, (unsigned)min(R, n_walk), &sc));
    __syncthreads();
    if (tid < m) bias[tid] = ord2f(bias_ord[tid]);
    __syncthreads();
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
    }
    __syncthreads();
    const float delta = delta_s, off = bias[j];
    const float inv = __fdiv_rn(1.0f, delta);
    const bool usual = delta >= QUANT_INV_MIN && delta <= 1.0f / QUANT_INV_MIN;  // uniform
    unsigned *out = reinterpret_cast<unsigned *>(qluts + (size_t)q * nprobe * entries);
    auto emit = [&](int p, float v) {
        // four neighbouring lanes' entries as one word (the lanes of a wavefront are at the same probe, or all beyond the last)
        const unsigned byte = usual ? quantize_entry_inv(v, off, delta, inv, (unsigned)nbins)
                                    : quantize_entry(v, off, delta, (unsigned)nbins);
        unsigned word = byte << (8 * (e & 3));
        word |= (unsigned)__builtin_amdgcn_mov_dpp((int)word, 0xB1, 0xf, 0xf, true);  // lanes 1 0 3 2
        word |= (unsigned)__builtin_amdgcn_mov_dpp((int)word, 0x4E, 0xf, 0xf, true);  // lanes 2 3 0 1
        if ((e & 3) == 0) out[((size_t)p * entries + e) >> 2] = word;
    };
#pragma unroll
    for (int k = 0; k < KEEP; ++k)
        if (sub + k * subs < nprobe) emit(sub + k * subs, kept[k]);  // uniform in a wavefront
    each_probe(KEEP * subs, emit);
}

// Calls of a few queries: Tables and the sums of the qmax walk in one launch.  Workgroup (p, q)
// builds the float tables of the query's p-th cell (the arithmetic of ivf_tables_kernel), leaves
// the minimum of each table, and computes the float ADC sums of the init codes that the walk takes from its list, with the tables still in LDS ...
constexpr int IVF_FRONT_NT = 256;

__global__ __launch_bounds__(IVF_FRONT_NT) void ivf_front_kernel(
    const float *__restrict__ codebooks, int d, int m, const float *__restrict__ queries,
    const float *__restrict__ coarse, const float *__restrict__ halves, const uint32_t *__restrict__ cell_ids,
    int Kh, const int32_t *__restrict__ probes, int nprobe, float *__restrict__ luts,
    const int64_t *__restrict__ list_off, const uint8_t *__restrict__ codes, int64_t n_total, int init,
    long long unit, unsigned *__restrict__ qunits, unsigned *__restrict__ cand,
    unsigned *__restrict__ mins, unsigned *__restrict__ nwalk_out)
{
    constexpr int NT = IVF_FRONT_NT;
    extern __shared__ double yr[];  // [d]
    __shared__ float lut_s[64 * 16];
    __shared__ unsigned long long wsum[NT / WAVE];
    __shared__ long long start_s[2], lo_s, total_s;
    __shared__ unsigned units_s;
    const int p = blockIdx.x, q = blockIdx.y;
    const int tid = threadIdx.x;
    const int dsub = d / m;
    const int entries = m * 16;
    const int B = m / 2;

    // geometry of the walk: list lengths one thread per probe, exclusive prefix sum
    static_assert(IVF_MAX_NPROBE <= NT, "one thread per probe");
    unsigned long long len = 0;
    long long my_lo = 0;
    if (tid == 0) units_s = 0;
    __syncthreads();
    if (tid < nprobe) {
        const int c = probes[(size_t)q * nprobe + tid];
        long long l = 0, h = 0;
        if (c >= 0) { l = list_off[c]; h = list_off[c + 1]; }
        if (l < 0 || h > n_total || h < l) l = h = 0;  // offsets that are not a list: nothing is read
        my_lo = l;
        len = (unsigned long long)(h - l);
        // units the scan kernel cuts this list into (the same expression as there)
        if (h > l) atomicAdd(&units_s, (unsigned)((h - l / 16 * 16 + unit - 1) / unit));
    }
    // this cell's residual while those loads travel
    const int cell = probes[(size_t)q * nprobe + p];
    if (cell >= 0) {
        if (coarse) {
            for (int t = tid; t < d; t += NT)
                yr[t] = (double)queries[(size_t)q * d + t] - (double)coarse[(size_t)cell * d + t];
        } else {  // list `cell` of a multi-index: the centroid is a pair of half-centroids
            const int dh = d >> 1;
            const unsigned id = cell_ids[cell];
            const float *h0 = halves + (size_t)(id / (unsigned)Kh) * dh;
            const float *h1 = halves + ((size_t)Kh + id % (unsigned)Kh) * dh;
            for (int t = tid; t < d; t += NT)
                yr[t] = (double)queries[(size_t)q * d + t] - (double)(t < dh ? h0[t] : h1[t - dh]);
        }
    }
    {
        const int l = lane_id();
        unsigned long long inc = len;
#pragma unroll
        for (int dd = 1; dd < WAVE; dd <<= 1) {
            const unsigned long long up = __shfl_up(inc, dd);
            if (l >= dd) inc += up;
        }
        if (l == WAVE - 1) wsum[tid / WAVE] = inc;
        __syncthreads();  // (also: the residual is complete)
        unsigned long long before = 0;
        for (int wv = 0; wv < tid / WAVE; ++wv) before += wsum[wv];
        if (tid == p) {
            start_s[0] = (long long)(before + inc - len);
            start_s[1] = (long long)(before + inc);
            lo_s = my_lo;
        }
        if (tid == nprobe - 1) total_s = (long long)(before + inc);
    }
    // Tables, Eq. (1) on the residual: float64 differences and sums, one rounding
    float *out = luts + ((size_t)q * nprobe + p) * entries;
    for (int e = tid; e < entries; e += NT) {
        float v = __builtin_inff();  // an unused probe slot: nothing of it is ever scanned
        if (cell >= 0) {
            const int j = e >> 4;
            const float *c = codebooks + (size_t)e * dsub;
            const double *y = yr + j * dsub;
            double acc = 0.0;
            for (int t = 0; t < dsub; ++t) {
                const double df = y[t] - (double)c[t];
                acc += df * df;
            }
            v = (float)acc;
        }
        out[e] = v;
        lut_s[e] = v;
    }
    __syncthreads();
    if (p == 0 && tid == 0) qunits[q] = units_s;
    // minimum of each table, as its order-preserving image
    if (tid < m) {
        unsigned mn = 0xffffffffu;
        for (int i = 0; i < 16; ++i) mn = min(mn, f2ord(lut_s[tid * 16 + i]));
        mins[((size_t)q * nprobe + p) * m + tid] = mn;
    }
    // the walk's codes that lie in this list: float32 sums in increasing j (as ivf_tables_kernel)
    const long long total = total_s;
    const int n_walk = (int)min((long long)init, total);
    {
        const long long s0 = start_s[0], s1 = min(start_s[1], (long long)n_walk);
        for (long long i = s0 + tid; i < s1; i += NT) {
            const unsigned *cw = reinterpret_cast<const unsigned *>(codes + (size_t)(lo_s + (i - s0)) * B);
            float acc = 0.0f;
            for (int k = 0; k < B / 4; ++k) {
                const unsigned w = cw[k];
                float e[8];
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const unsigned comps = (w >> (8 * b)) & 0xffu;
                    const int jb = 4 * k + b;
                    e[2 * b] = lut_s[(2 * jb) * 16 + (comps & 15u)];
                    e[2 * b + 1] = lut_s[(2 * jb + 1) * 16 + (comps >> 4)];
                }
#pragma unroll
                for (int b = 0; b < 8; ++b) acc = acc + e[b];
            }
            cand[(size_t)q * QADC_MAX_INIT + i] = f2ord(acc);
        }
    }
    if (p == 0 && tid == 0) nwalk_out[q] = (unsigned)n_walk;
}

// ... then one workgroup per query selects qmax among the sums, joins the minima of the tables into
// the biases and derives delta: the arithmetic of quantize_luts_kernel.  (A launch of its own: the
// kernel boundary makes the sums visible; a count of finished workgroups with memory fences, tried
// first, made every workgroup of the launch before write the L2 back.)
constexpr int IVF_FINISH_NT = 1024;

__global__ __launch_bounds__(IVF_FINISH_NT) void ivf_finish_kernel(
    const unsigned *__restrict__ cand, const unsigned *__restrict__ mins, const unsigned *__restrict__ nwalk,
    int nprobe, int m, int R, int nbins, int qmin_mode, float *__restrict__ qmax_out,
    float *__restrict__ qbias, float *__restrict__ qdelta)
{
    constexpr int NT = IVF_FINISH_NT;
    __shared__ unsigned cand_s[QADC_MAX_INIT];
    __shared__ float bias_s[64];
    __shared__ unsigned bias_ord[64];
    __shared__ SelectScratch sc;
    const int q = blockIdx.x;
    const int tid = threadIdx.x;
    const int n_walk = (int)nwalk[q];
    for (int i = tid; i < n_walk; i += NT) cand_s[i] = cand[(size_t)q * QADC_MAX_INIT + i];
    for (int e = tid; e < m; e += NT) bias_ord[e] = 0xffffffffu;
    __syncthreads();
    for (int e = tid; e < nprobe * m; e += NT)  // (m divides NT: a thread meets the same table every round)
        atomicMin(&bias_ord[e % m], mins[(size_t)q * nprobe * m + e]);
    __syncthreads();
    if (tid < m) bias_s[tid] = ord2f(bias_ord[tid]);
    __syncthreads();
    float qmax = 0.0f;  // (no code in the probed lists)
    if (n_walk > 0)     // uniform
        qmax = ord2f(block_radix_select<unsigned, 4>(cand_s, (unsigned)n_walk, (unsigned)min(R, n_walk), &sc));
    if (tid == 0) {
        float qmin;
        if (qmin_mode == QADC_QMIN_GLOBAL) {
            qmin = bias_s[0];
            for (int j = 1; j < m; ++j) qmin = fminf(qmin, bias_s[j]);
            for (int j = 0; j < m; ++j) bias_s[j] = qmin;
        } else {
            qmin = 0.0f;
            for (int j = 0; j < m; ++j) qmin = qmin + bias_s[j];
        }
        float delta = __fdiv_rn(qmax - qmin, (float)nbins);
        if (!(delta > 0.0f)) delta = 1.0f;
        qdelta[q] = delta;
        qmax_out[q] = qmax;
    }
    __syncthreads();
    if (tid < m) qbias[(size_t)q * m + tid] = bias_s[tid];
}

// ------------------------------------------------------------------- Seed
//
// A bound for the scan: the quantized sums (Alg. 2) of a sample of the query's codes -- the
// first `per_list` codes of the closest lists and those of the qmax walk -- are histogrammed by one workgroup per query;
// the bin where the running count reaches R bounds the query's R-th smallest sum from above.
// It is left in the first word of the query's control block as bound + 1 (0: no bound).
// The sample uses the 16-entry tables directly (two lookups per code byte): building pair
// tables for every cell would cost more than the sample itself.
constexpr int IVF_SEED_NT = 1024;
constexpr int IVF_SEED_PROBES = 16;  // closest cells whose lists are sampled
constexpr int IVF_SEED_PCH = 32;  // probed cells whose tables are in LDS at a time

// What the shared-list scan starts from (cnt null: there is none): the pairs of every cell, the queries' bounds and flags.
struct IvfPairs {
    unsigned *cnt, *taus, *flags;
    int K;
};

template <int B>
__global__ __launch_bounds__(IVF_SEED_NT) void ivf_seed_kernel(
    const int64_t *__restrict__ list_off, const uint8_t *__restrict__ codes,
    const int32_t *__restrict__ probes, int nprobe, const uint8_t *__restrict__ qluts, int cap_i,
    int R, int per_list, char *__restrict__ ws, size_t ws_stride, int64_t n_total, int long_shift, int nseed, int init,
    IvfQuantizer fq, IvfPairs pairs)
{
    constexpr int NT = IVF_SEED_NT;
    constexpr int TAB = 2 * B * 16;  // bytes of one cell's quantized tables
    __shared__ __attribute__((aligned(16))) uint8_t tab[IVF_SEED_PCH * TAB];
    __shared__ long long lo[IVF_MAX_NPROBE];
    __shared__ int len[IVF_MAX_NPROBE];
    __shared__ int more[IVF_MAX_NPROBE];  // codes sampled beyond per_list (long lists, long_shift > 0)
    __shared__ unsigned hist[256];
    const int tid = threadIdx.x;
    const int q = blockIdx.x;
    // a few queries: the probed lists of a query are split over gridDim.y workgroups, which add
    // their histograms into the query's control block
    const int parts = gridDim.y;
    // (nseed <= nprobe: only the lists of the nseed closest cells are sampled)
    const int per_part = (nseed + parts - 1) / parts;
    const int p_begin = blockIdx.y * per_part, p_end = min(nseed, p_begin + per_part);
    const unsigned cap = (unsigned)cap_i;
    long long whole = 0;
    if (tid < nprobe) {
        const int cell = probes[(size_t)q * nprobe + tid];
        long long l = 0, h = 0;
        if (cell >= 0) { l = list_off[cell]; h = list_off[cell + 1]; }
        if (l < 0 || h > n_total || h < l) l = h = 0;  // offsets that are not a list: nothing is read
        lo[tid] = l;
        whole = h - l;
        len[tid] = (int)min((long long)per_list, whole);
    }
    // The sample holds the codes that qmax was found among: R of them are within the quantizer's range (sums that saturate do
    // not count: next to always fewer than leave R), so that there is a bound.  Where it did not, lists longer than
    // per_list and many init codes left fewer than R: no bound, and a scan with barriers in every tile.  (100 queries x 100 lists
    // of 3900 codes, m = 16, R = 100, 3000 init codes 366 -> 148 us a call; 500 x 64 of 500, m = 8, 1000 init codes 389 -> 173.)
    // With long_shift the sample of a list is at least its 2^-long_shift part: the bound then reflects the lists in
    // proportion to their lengths.
    long long least = 0;
    if (tid < WAVE) {  // (the closest 64 at most; nseed is 16)
        const unsigned taken = tid < nseed ? (unsigned)min((long long)init, whole) : 0u;
        least = max(0, init - (int)(wave_running_sum(taken) - taken));  // what the walk still takes when it comes to this list
    }
    if (long_shift > 0) least = max(least, min(whole >> long_shift, 1ll << 30));
    if (tid < nprobe) more[tid] = (int)max(0ll, min(least, whole) - per_list);
    for (int e = tid; e < 256; e += NT) hist[e] = 0;
    for (int p0 = p_begin; p0 < p_end; p0 += IVF_SEED_PCH) {  // uniform
        const int np = min(IVF_SEED_PCH, p_end - p0);
        __syncthreads();  // geometry and histogram ready; nobody still reads the previous tables
        if (fq.luts) {  // uniform
            const float *src = fq.luts + ((size_t)q * nprobe + p0) * TAB;
            const float delta = fq.delta[q];
            for (int e = tid; e < np * (TAB / 4); e += NT)
                reinterpret_cast<unsigned *>(tab)[e] =
                    quantize_word(src + (size_t)(e / (TAB / 4)) * TAB, e % (TAB / 4),
                                  fq.bias + (size_t)q * (2 * B), delta, cap);
        } else {
            const unsigned *src = reinterpret_cast<const unsigned *>(qluts + ((size_t)q * nprobe + p0) * TAB);
            for (int e = tid; e < np * (TAB / 4); e += NT) reinterpret_cast<unsigned *>(tab)[e] = src[e];
        }
        __syncthreads();
        for (int i = tid; i < np * per_list; i += NT) {
            const int pp = i / per_list, c = i - pp * per_list;
            if (c >= len[p0 + pp]) continue;
            const unsigned *cw = reinterpret_cast<const unsigned *>(codes + (size_t)(lo[p0 + pp] + c) * B);
            const uint8_t *t = tab + pp * TAB;
            unsigned sum = 0;
#pragma unroll
            for (int k = 0; k < B / 4; ++k) {
                const unsigned x = cw[k];
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const unsigned v = (x >> (8 * b)) & 0xffu;
                    const int jb = 4 * k + b;
                    sum += (unsigned)t[(2 * jb) * 16 + (v & 15u)] + (unsigned)t[(2 * jb + 1) * 16 + (v >> 4)];
                }
            }
            if (sum < cap) atomicAdd(&hist[sum], 1u);  // saturated sums carry no information
        }
        for (int pp = 0; pp < np; ++pp) {  // uniform
            const int extra = more[p0 + pp];
            const uint8_t *t = tab + pp * TAB;
            for (int c = per_list + tid; c < per_list + extra; c += NT) {
                const unsigned *cw = reinterpret_cast<const unsigned *>(codes + (size_t)(lo[p0 + pp] + c) * B);
                unsigned sum = 0;
#pragma unroll
                for (int k = 0; k < B / 4; ++k) {
                    const unsigned x = cw[k];
#pragma unroll
                    for (int b = 0; b < 4; ++b) {
                        const unsigned v = (x >> (8 * b)) & 0xffu;
                        const int jb = 4 * k + b;
                        sum += (unsigned)t[(2 * jb) * 16 + (v & 15u)] + (unsigned)t[(2 * jb + 1) * 16 + (v >> 4)];
                    }
                }
                if (sum < cap) atomicAdd(&hist[sum], 1u);
            }
        }
    }
    __syncthreads();
    ScanHeader *hdr = reinterpret_cast<ScanHeader *>(ws + (size_t)q * ws_stride);
    if (parts > 1) {
        // ghist[1][bin]: the query's histogram over all parts; every workgroup of the scan kernel derives
        // the bound from it (the launch boundary orders the two; no count of finished parts, no fences)
        if (tid < 256 && hist[tid])
            __hip_atomic_fetch_add(&hdr->ghist[1][tid], hist[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;  // uniform
    }
    if (tid < WAVE) {
        unsigned h[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) h[b] = hist[4 * tid + b];
        const unsigned t = wave_threshold_bin<4>(h, (unsigned)R);
        if (tid == 0) {
            hdr->ghist[0][0] = (t < 256u) ? t + 1u : 0u;
            if (pairs.cnt) {
                pairs.taus[q] = (t < 256u) ? t : IVFS_NONE;
                pairs.flags[q] = (t < 256u) ? 2u : 1u;  // 2: shared lists there, the others by the per-query kernel; 1: all by that one
            }
        }
    }
    if (pairs.cnt && tid < nprobe) {
        const int cell = probes[(size_t)q * nprobe + tid];
        if (cell >= 0 && cell < pairs.K) atomicAdd(&pairs.cnt[cell], 1u);
    }
}

// ------------------------------------------------------------------- Scan

constexpr int IVF_MAP_NT = 1024;
constexpr int IVF_MAP_MAXQ = 4096;   // queries per batch, at most
constexpr unsigned IVF_NO_WG = 0xffffffffu;  // (no entry of the map: units_per_wg is below 256)
constexpr int IVF_MAX_UNITS = 255;
constexpr unsigned long long IVF_FILL_WGS = 4096;

// Workgroups of the scan: query q gets W_q = clamp(ceil(units_q / units_per_wg), 1, Wmax) of them, work in proportion to
// the lists it probes.  wgmap[b] = (units_per_wg - 1) << 24 | q << 12 | g for workgroup b of the grid, IVF_NO_WG beyond
// the last one.  nb <= IVF_MAP_MAXQ, Wmax <= 4096.
// units_per_wg: as many as leave IVF_FILL_WGS workgroups, at most max_units.  (Always 16: the 300
// workgroups of 150 queries over 1e6 codes walked 16 units each one after the other, 130 us; 52 with as many as the GPU holds.
// 64 queries over 4e6 codes 239 -> 165 us per call; 1024, 2048 and 8192 workgroups: up to 8, 4 and 9 % slower.)
// With `flags`, a query whose flag is not 1 is scanned over its other set of cells (see ivf_scan_kernel)
// and its units are qunits_alt's.
// Queries with more than the average number of units come first in the grid.  Every workgroup takes the running sums over all
// queries and fills its share of the map: 5 us (one workgroup that also ordered the queries by their units 8 to 20; in the
// order of the queries alone the scan took 3 to 6 % longer).
__global__ __launch_bounds__(IVF_MAP_NT) void ivf_wgmap_kernel(const unsigned *__restrict__ qunits, int nb,
                                                              int max_units, int Wmax,
                                                              unsigned *__restrict__ wgmap,
                                                              const unsigned *__restrict__ qunits_alt,
                                                              const unsigned *__restrict__ flags)
{
    constexpr int PER = IVF_MAP_MAXQ / IVF_MAP_NT;  // queries per thread, neighbours
    __shared__ unsigned start[2][IVF_MAP_MAXQ];     // first workgroup of query q, or of those behind it
    __shared__ unsigned total_s;
    __shared__ unsigned long long usum[IVF_MAP_NT / WAVE];
    __shared__ unsigned wsum[2][IVF_MAP_NT / WAVE];
    const int tid = threadIdx.x, l = lane_id();
    unsigned un[PER];
    unsigned long long all = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int q = tid * PER + k;
        un[k] = q < nb ? ((flags && flags[q] != 1u) ? qunits_alt[q] : qunits[q]) : 0u;
        all += un[k];
    }
#pragma unroll
    for (int w = 32; w >= 1; w >>= 1) all += __shfl_xor(all, w);
    if (l == 0) usum[tid / WAVE] = all;
    __syncthreads();
    all = 0;
    for (int w = 0; w < IVF_MAP_NT / WAVE; ++w) all += usum[w];
    const int units_per_wg = (int)max(1ull, min((unsigned long long)max_units, all / IVF_FILL_WGS));
    // running sums of the workgroups, those of the queries with more than the average number of units apart: they come first
    const unsigned average = (unsigned)(all / (unsigned long long)nb);
    unsigned mine[2] = {0, 0}, cls[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        cls[k] = un[k] > average ? 0u : 1u;
        un[k] = tid * PER + k < nb ? min((unsigned)Wmax, max(1u, (un[k] + (unsigned)units_per_wg - 1u) / (unsigned)units_per_wg)) : 0u;
        mine[0] += cls[k] == 0u ? un[k] : 0u;
        mine[1] += cls[k] == 1u ? un[k] : 0u;
    }
    unsigned inc[2] = {mine[0], mine[1]};
#pragma unroll
    for (int dd = 1; dd < WAVE; dd <<= 1) {
        const unsigned up0 = __shfl_up(inc[0], dd), up1 = __shfl_up(inc[1], dd);
        if (l >= dd) { inc[0] += up0; inc[1] += up1; }
    }
    if (l == WAVE - 1) { wsum[0][tid / WAVE] = inc[0]; wsum[1][tid / WAVE] = inc[1]; }
    __syncthreads();
    unsigned at[2] = {inc[0] - mine[0], inc[1] - mine[1]}, first = 0;
    for (int w = 0; w < IVF_MAP_NT / WAVE; ++w) {
        if (w < tid / WAVE) { at[0] += wsum[0][w]; at[1] += wsum[1][w]; }
        first += wsum[0][w];
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        // (a query takes no room among those of the other kind)
        const int q = tid * PER + k;
        start[0][q] = at[0];
        start[1][q] = first + at[1];
        at[cls[k]] += un[k];
    }
    if (tid == IVF_MAP_NT - 1) total_s = first + at[1];
    __syncthreads();
    const unsigned total = total_s;
    const unsigned slots = (unsigned)nb * (unsigned)Wmax;
    for (unsigned b = blockIdx.x * IVF_MAP_NT + tid; b < slots; b += gridDim.x * IVF_MAP_NT) {
        unsigned v = IVF_NO_WG;
        if (b < total) {
            const unsigned *s = start[b < first ? 0 : 1];
            int lo_q = 0, hi_q = nb;  // last query whose first workgroup is <= b
            while (hi_q - lo_q > 1) {
                const int mid = (lo_q + hi_q) >> 1;
                if (s[mid] <= b) lo_q = mid; else hi_q = mid;
            }
            v = ((unsigned)(units_per_wg - 1) << 24) | ((unsigned)lo_q << 12) | (b - s[lo_q]);
        }
        wgmap[b] = v;
    }
}


// (In 64 bits the lists' geometry took 4 KiB more, a workgroup less per compute unit: 150 queries over 1e6 codes 108 against
// 102 us per call, 350 over 8e6 265 against 245.)
struct IvfShared {
    SelectScratch sel;
    unsigned ccnt;
    unsigned tcnt[3];
    unsigned tau;
    unsigned fcnt;                         // append counter of the barrier-free pass
    unsigned wsum[1024 / WAVE];           // unit counts of the wavefronts (prefix sum)
    unsigned ustart[IVF_MAX_NPROBE + 1];  // units before probe p (positions and units are below 2^32)
    unsigned a0[IVF_MAX_NPROBE];          // list start rounded down to 16 codes
    unsigned lo[IVF_MAX_NPROBE];
    unsigned hi[IVF_MAX_NPROBE];
};

// NT threads per workgroup: IVF_NT for batches; 1024 for a few queries, whose lists must be read
// by few workgroups at once (a workgroup has one tile in flight and the next one requested).
template <int B, int NT>
__global__ __launch_bounds__(NT) void ivf_scan_kernel(
    const int64_t *__restrict__ list_off, const uint8_t *__restrict__ codes, int64_t n_total,
    const int32_t *__restrict__ probes, int nprobe, const uint8_t *__restrict__ qluts, int cap_i,
    int R, int units_per_wg, int Wmax, const unsigned *__restrict__ wgmap, char *__restrict__ ws,
    size_t ws_stride, size_t counts_off, size_t lists_off, const int32_t *__restrict__ probes_alt,
    const unsigned *__restrict__ flags, IvfQuantizer fq, int hist_bound)
{
    using C = ScanCfg<B, NT>;
    constexpr long long UNIT = (long long)IVF_UNIT_TILES * IVF_NT * C::CPT;  // the same codes whatever NT
    static_assert(UNIT % C::TILE == 0, "whole tiles per unit");
    // without a map (a few queries): Wmax workgroup slots per query, in query order
    const unsigned me = wgmap ? wgmap[blockIdx.x]
                              : ((blockIdx.x / (unsigned)Wmax) << 12) | (blockIdx.x % (unsigned)Wmax);  // uniform
    if (me == IVF_NO_WG) return;
    __shared__ __attribute__((aligned(16))) uint8_t ptab[B * 256];
    __shared__ __attribute__((aligned(16))) uint8_t qlut_s[2 * B * 16];
    __shared__ uint64_t keys[C::CAP];
    __shared__ IvfShared sh;

    const int tid = threadIdx.x;
    const int q = (int)((me >> 12) & 4095u);
    const int g = (int)(me & 4095u);
    if (wgmap) units_per_wg = (int)(me >> 24) + 1;  // (uniform)
    const unsigned cap = (unsigned)cap_i;
    // bound + 1 left by the seed kernel (uniform load), 0 when there is none; hist_bound: the seed
    // kernel's workgroups left the query's histogram instead, and the bound is derived below
    const ScanHeader *hdr_in = reinterpret_cast<const ScanHeader *>(ws + (size_t)q * ws_stride);
    unsigned tau1 = hist_bound ? 0u : hdr_in->ghist[0][0];
    unsigned hb[4] = {0, 0, 0, 0};
    if (hist_bound && tid < WAVE) {
        const uint4 v = *reinterpret_cast<const uint4 *>(&hdr_in->ghist[1][4 * tid]);
        hb[0] = v.x; hb[1] = v.y; hb[2] = v.z; hb[3] = v.w;
    }

    // Geometry of the probed lists, one thread per probe, then an exclusive prefix sum of the
    // unit counts.
    static_assert(IVF_MAX_NPROBE <= NT, "one thread per probe");
    unsigned my_units = 0;
    // (with flags: a query whose flag is not 1 leaves some of its cells to the shared-list scan and
    // takes the others, probes_alt, here; the tables stay indexed by the slot)
    const int32_t *pr = (flags && flags[q] != 1u) ? probes_alt : probes;  // uniform
    if (tid < nprobe) {
        const int cell = pr[(size_t)q * nprobe + tid];
        long long l = 0, h = 0;
        if (cell >= 0) { l = list_off[cell]; h = list_off[cell + 1]; }
        if (l < 0 || h > n_total || h < l) l = h = 0;  // offsets that are not a list: nothing is read
        const long long a = l / 16 * 16;
        sh.lo[tid] = (unsigned)l;
        sh.hi[tid] = (unsigned)h;
        sh.a0[tid] = (unsigned)a;
        my_units = (h > l) ? (unsigned)((h - a + UNIT - 1) / UNIT) : 0u;
    }
    {
        const int l = lane_id();
        const unsigned inc = wave_running_sum(my_units);
        if (l == WAVE - 1) sh.wsum[tid / WAVE] = inc;
        __syncthreads();
        unsigned before = 0;
        for (int wv = 0; wv < tid / WAVE; ++wv) before += sh.wsum[wv];
        if (tid < nprobe) sh.ustart[tid] = before + inc - my_units;
        if (tid == nprobe - 1) sh.ustart[nprobe] = before + inc;
        if (tid == 0) { sh.tcnt[0] = 0; sh.fcnt = 0; }
    }
    if (hist_bound && tid < WAVE) {  // the bin where the running count of the sample reaches R
        const unsigned t = wave_threshold_bin<4>(hb, (unsigned)R);
        if (tid == 0) sh.tau = (t < 256u) ? t + 1u : 0u;
    }
    for (int e = tid; e < 256; e += NT) sh.sel.hist[e] = 0;
    __syncthreads();
    if (hist_bound) tau1 = sh.tau;  // uniform
    const long long units = sh.ustart[nprobe];
    // Workgroups of this query: in proportion to its work (a query whose cell is one of the few
    // huge lists gets up to Wmax of them, a query of short lists a handful) -- the count the
    // map kernel derived from the same number of units.
    const int W = (int)min((long long)Wmax, max(1ll, (units + units_per_wg - 1) / units_per_wg));
    if (g >= W) return;  // uniform; with a map it cannot happen

    uint64_t lim = ~0ull;  // keys >= lim cannot be among the R best of this workgroup's codes
    unsigned have = 0;
    int rot = 0;
    int cur_p = -1;
    bool first_tile = true;
    const long long ub = units * g / W, ue = units * (g + 1) / W;

    // probe of unit u (binary search, same result in every thread)
    auto probe_of = [&](long long u) {
        int lo_p = 0, hi_p = nprobe;
        while (hi_p - lo_p > 1) {
            const int mid = (lo_p + hi_p) >> 1;
            if (sh.ustart[mid] <= u) lo_p = mid; else hi_p = mid;
        }
        return lo_p;
    };
    // pair tables of probe p (called by the whole workgroup)
    auto load_tables = [&](int p) {
        __syncthreads();  // nobody still reads the previous pair tables
        if (fq.luts) {  // uniform
            const float *lt = fq.luts + ((size_t)q * nprobe + p) * (2 * B) * 16;
            const float delta = fq.delta[q];
            for (int e = tid; e < 2 * B * 4; e += NT)
                reinterpret_cast<unsigned *>(qlut_s)[e] =
                    quantize_word(lt, e, fq.bias + (size_t)q * (2 * B), delta, cap);
        } else {
            const uint8_t *qlut = qluts + ((size_t)q * nprobe + p) * (2 * B) * 16;
            for (int e = tid; e < 2 * B * 4; e += NT)
                reinterpret_cast<unsigned *>(qlut_s)[e] = reinterpret_cast<const unsigned *>(qlut)[e];
        }
        __syncthreads();
        pair_rows_from_lds<B, NT>(qlut_s, cap, ptab);
        __syncthreads();
    };

    // With a bound: no barrier inside a unit.  The bound is below the saturation value, so a
    // sum that passes needs no clamp; the append code only runs in waves with a hit.  After
    // each unit the list is looked at: the nearest cells hold most of a query's candidates, so
    // the workgroups that scan them cut their list back to its R smallest keys (which tightens
    // their own bound) whenever it grows.  Should the list overflow inside a unit, everything
    // is redone by the careful pass below.
    bool careful = true;
    if (tau1 != 0u) {
        careful = false;
        lim = (uint64_t)tau1 << 32;  // keys with sum <= bound
        for (long long u = ub; u < ue; ++u) {  // uniform
            const int p = probe_of(u);
            const long long lo = sh.lo[p], hi = sh.hi[p];
            const long long u0 = sh.a0[p] + (u - sh.ustart[p]) * UNIT;
            const long long u1 = min(hi, u0 + UNIT);
            // The next tile of the unit is requested before the current one is used; on a change of
            // list the new tables are requested first and the unit's first tile right behind them
            // (loads return in the order they were issued), so the tile travels while the pair
            // tables are rebuilt.
            uint4 w[2], wn[2];
            int nc[2], ncn[2];
            const bool new_list = p != cur_p;  // uniform
            // a row of a pair table per thread: the 16 entries of its even table, one entry of the odd one
            constexpr int ROWS = (B * 16 + NT - 1) / NT;
            uint4 low[ROWS];
            unsigned high[ROWS];
            float4 fword = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (new_list) {
                if (fq.luts) {  // uniform
                    if (tid < 2 * B * 4)
                        fword = reinterpret_cast<const float4 *>(fq.luts + ((size_t)q * nprobe + p) * (2 * B) * 16)[tid];
                } else {
                    const uint8_t *ql = qluts + ((size_t)q * nprobe + p) * (2 * B) * 16;
#pragma unroll
                    for (int r = 0; r < ROWS; ++r) {
                        const int e = min(tid + r * NT, B * 16 - 1);
                        low[r] = *reinterpret_cast<const uint4 *>(ql + (e >> 4) * 32);
                        high[r] = ql[(e >> 4) * 32 + 16 + (e & 15)];
                    }
                }
            }
            asm volatile("" ::: "memory");
            tile_load<B, NT>(codes, u0, n_total, wn, ncn);
            asm volatile("" ::: "memory");
            if (new_list) {
                __syncthreads();  // nobody still reads the previous pair tables
                if (fq.luts) {    // uniform
                    if (tid < 2 * B * 4) {  // the query's quantizer applied to the four entries
                        const float b = fq.bias[(size_t)q * (2 * B) + (tid >> 2)];
                        const float delta = fq.delta[q];
                        reinterpret_cast<unsigned *>(qlut_s)[tid] =
                            quantize_entry(fword.x, b, delta, cap) | (quantize_entry(fword.y, b, delta, cap) << 8) |
                            (quantize_entry(fword.z, b, delta, cap) << 16) | (quantize_entry(fword.w, b, delta, cap) << 24);
                    }
                    __syncthreads();
                    pair_rows_from_lds<B, NT>(qlut_s, cap, ptab);
                } else {
#pragma unroll
                    for (int r = 0; r < ROWS; ++r)
                        if (tid + r * NT < B * 16)
                            reinterpret_cast<uint4 *>(ptab)[tid + r * NT] = pair_row(low[r], high[r], cap);
                }
                __syncthreads();
                cur_p = p;
            }
            for (long long t0 = u0; t0 < u1; t0 += C::TILE) {
                w[0] = wn[0]; w[1] = wn[1];
                nc[0] = ncn[0]; nc[1] = ncn[1];
                if (t0 + C::TILE < u1) tile_load<B, NT>(codes, t0 + C::TILE, n_total, wn, ncn);  // uniform
                // Sums only; positions, validity and keys are worked out in the wavefronts that hold a
                // sum small enough to pass (a slot without a code may hold one too: it is dropped there).
                // Entries are not negative, so a code whose first half of the bytes already sums to more
                // than a passing sum may cannot pass: only the lanes that hold a code still in the race
                // look up the other half (a wavefront without one skips it; with few lanes left they no
                // longer collide on the LDS banks), the others keep their partial sum.
                // a key below lim has a sum of at most (lim - 1) >> 32
                const unsigned limsum = (unsigned)((lim - 1ull) >> 32);
                unsigned sm[C::CPT];
                if constexpr (B <= 16) {
                    constexpr int CPV = 16 / B;
                    // stages of bytes, a check after each but the last
                    constexpr int NS = QADC_IVF_EARLY_STAGES(B);
                    constexpr int cut[4] = {0, NS == 3 ? B / 4 : (NS == 2 ? B / 2 : B), NS == 3 ? B / 2 : B, B};
#pragma unroll
                    for (int c = 0; c < 2 * CPV; ++c) sm[c] = 0;
                    bool go = true;
#pragma unroll
                    for (int st = 0; st < NS; ++st) {
                        if (go) {
                            unsigned part = 0xffffffffu;
#pragma unroll
                            for (int v = 0; v < 2; ++v) {
#pragma unroll
                                for (int c = 0; c < CPV; ++c) {
                                    unsigned s = sm[v * CPV + c];
#pragma unroll
                                    for (int jb = cut[st]; jb < cut[st + 1]; ++jb)
                                        s += ptab[jb * 256 + byte_of(w[v], c * B + jb)];
                                    sm[v * CPV + c] = s;
                                    part = min(part, s);
                                }
                            }
                            go = part <= limsum;
                        }
                    }
                } else {
                    unsigned s = 0;
#pragma unroll
                    for (int jb = 0; jb < 16; ++jb) s += ptab[jb * 256 + byte_of(w[0], jb)];
                    if (s <= limsum) {
#pragma unroll
                        for (int jb = 16; jb < 32; ++jb) s += ptab[jb * 256 + byte_of(w[1], jb & 15)];
                    }
                    sm[0] = s;
                }
                unsigned best = sm[0];
#pragma unroll
                for (int c = 1; c < C::CPT; ++c) best = min(best, sm[c]);
                if (__ballot(best <= limsum) != 0ull) {
#pragma unroll
                    for (int c = 0; c < C::CPT; ++c) {
                        long long pos;
                        bool valid;
                        if constexpr (B <= 16) {
                            constexpr int CPV = 16 / B;
                            const int v = c / CPV, cc = c % CPV;
                            pos = t0 + (long long)((v * NT + tid) * CPV + cc);
                            valid = (cc < nc[v]) && pos >= lo && pos < u1;
                        } else {
                            pos = t0 + tid;
                            valid = nc[0] && pos >= lo && pos < u1;
                        }
                        const uint64_t key = ((uint64_t)sm[c] << 32) | (uint64_t)pos;
                        const bool pass = valid && key < lim;
                        const unsigned slot = wave_append_slot(pass, &sh.fcnt);
                        if (pass && slot < (unsigned)C::CAP) keys[slot] = key;
                    }
                }
            }
            __syncthreads();
            have = sh.fcnt;
            __syncthreads();  // everybody has read the count before the next unit bumps it
            if (have > (unsigned)C::CAP) { careful = true; break; }  // uniform: keys were dropped
            // cut the list back once it holds more than R keys and has grown past half its slack
            // (a list of at most R keys is the workgroup's result so far: nothing to drop)
            if (have > max((unsigned)R, (unsigned)SCAN_SLACK / 2)) {
                const uint64_t kth = compact_candidates<uint64_t, 5, NT, C::CAP>(
                    keys, have, (unsigned)R, &sh.sel, &sh.ccnt);
                lim = min(lim, kth + 1ull);
                have = (unsigned)R;
                if (tid == 0) sh.fcnt = (unsigned)R;
                __syncthreads();
            }
        }
        if (careful) { have = 0; cur_p = -1; lim = ~0ull; }
    }

    // Careful pass.  Workgroup g takes a contiguous range of the query's units: consecutive
    // units mostly belong to the same list, so the pair tables are rebuilt only when the list
    // changes.
    for (long long u = ub; careful && u < ue; ++u) {  // uniform
        const int p = probe_of(u);
        if (p != cur_p) { load_tables(p); cur_p = p; }
        const long long lo = sh.lo[p], hi = sh.hi[p];
        const long long u0 = sh.a0[p] + (u - sh.ustart[p]) * UNIT;
        const long long u1 = min(hi, u0 + UNIT);
        for (long long t0 = u0; t0 < u1; t0 += C::TILE) {
            unsigned *ctr = &sh.tcnt[rot];
            const int nxt = (rot == 2) ? 0 : rot + 1;
            if (tid == 0) sh.tcnt[nxt] = 0;
            uint4 w[2];
            int nc[2];
            tile_load<B, NT>(codes, t0, n_total, w, nc);  // may reach into the neighbouring lists
            uint64_t k[C::CPT];
            if constexpr (B <= 16) {
                constexpr int CPV = 16 / B;
#pragma unroll
                for (int v = 0; v < 2; ++v) {
#pragma unroll
                    for (int c = 0; c < CPV; ++c) {
                        unsigned s = 0;
#pragma unroll
                        for (int jb = 0; jb < B; ++jb) s += ptab[jb * 256 + byte_of(w[v], c * B + jb)];
                        s = min(s, cap);
                        const long long pos = t0 + (long long)((v * NT + tid) * CPV + c);
                        const bool valid = (c < nc[v]) && pos >= lo && pos < u1;
                        k[v * CPV + c] = valid ? (((uint64_t)s << 32) | (uint64_t)pos) : ~0ull;
                    }
                }
            } else {
                unsigned s = 0;
#pragma unroll
                for (int jb = 0; jb < 32; ++jb) s += ptab[jb * 256 + byte_of(w[jb >> 4], jb & 15)];
                s = min(s, cap);
                const long long pos = t0 + tid;
                const bool valid = nc[0] && pos >= lo && pos < u1;
                k[0] = valid ? (((uint64_t)s << 32) | (uint64_t)pos) : ~0ull;
            }

            if (first_tile) {
                // bound the workgroup's share by its own first tile: the bin of the R-th
                // smallest unsaturated sum (keys above it cannot be among the R best)
#pragma unroll
                for (int c = 0; c < C::CPT; ++c)
                    if (k[c] != ~0ull && (unsigned)(k[c] >> 32) < cap)
                        atomicAdd(&sh.sel.hist[(unsigned)(k[c] >> 32)], 1u);
                __syncthreads();
                if (tid < WAVE) {
                    const int l = tid;
                    unsigned h0 = sh.sel.hist[4 * l], h1 = sh.sel.hist[4 * l + 1];
                    unsigned h2 = sh.sel.hist[4 * l + 2], h3 = sh.sel.hist[4 * l + 3];
                    const unsigned tot = h0 + h1 + h2 + h3;
                    unsigned inc = tot;
#pragma unroll
                    for (int dd = 1; dd < WAVE; dd <<= 1) {
                        const unsigned up = __shfl_up(inc, dd);
                        if (l >= dd) inc += up;
                    }
                    const unsigned long long mm = __ballot(inc >= (unsigned)R);
                    unsigned t = cap;
                    if (mm) {
                        const int fl = __ffsll((long long)mm) - 1;
                        unsigned run = inc - tot, bin = 4u * l + 3u;
                        const unsigned hh[4] = {h0, h1, h2, h3};
                        bool found = false;
#pragma unroll
                        for (int b = 0; b < 4; ++b) {
                            run += hh[b];
                            if (!found && run >= (unsigned)R) { bin = 4u * l + b; found = true; }
                        }
                        t = __shfl(bin, fl);
                    }
                    if (tid == 0) sh.tau = min(t, cap);
                }
                __syncthreads();
                lim = ((uint64_t)sh.tau + 1ull) << 32;
                first_tile = false;
            }

            uint64_t best = k[0];
#pragma unroll
            for (int c = 1; c < C::CPT; ++c) best = min(best, k[c]);
            if (__ballot(best < lim) != 0ull) {  // the append code only runs in waves with a hit
#pragma unroll
                for (int c = 0; c < C::CPT; ++c) {
                    const bool pass = k[c] < lim;
                    const unsigned slot = have + wave_append_slot(pass, ctr);
                    if (pass) keys[slot] = k[c];
                }
            }
            __syncthreads();
            have += *ctr;
            rot = nxt;
            if (have > (unsigned)SCAN_SLACK) {
                const uint64_t kth = compact_candidates<uint64_t, 5, NT, C::CAP>(
                    keys, have, (unsigned)R, &sh.sel, &sh.ccnt);
                lim = min(lim, kth + 1ull);
                have = (unsigned)R;
            }
        }
    }

    if (have > (unsigned)R) {
        compact_candidates<uint64_t, 5, NT, C::CAP>(keys, have, (unsigned)R, &sh.sel, &sh.ccnt);
        have = (unsigned)R;
    }
    if (have == 0) return;
    unsigned *counts = reinterpret_cast<unsigned *>(ws + (size_t)q * ws_stride + counts_off);
    uint64_t *dst = reinterpret_cast<uint64_t *>(ws + (size_t)q * ws_stride + lists_off) + (size_t)g * R;
    if (tid == 0) counts[g] = have;
    for (unsigned i = tid; i < have; i += NT) dst[i] = keys[i];
}

// Cells given by the caller: a cell outside [0, K) and a cell that an earlier slot of the same
// query already names become unused slots (-1) -- a list is scanned once, so that keys stay
// unique, and nothing outside list_off is read.
__global__ __launch_bounds__(256) void ivf_take_probes_kernel(const int32_t *__restrict__ in, int nprobe, int K, int64_t total,
                                       int32_t *__restrict__ probes, IvfClear clr, int nq)
{
    if (clr.scan_ws && (int)blockIdx.x < nq) {  // uniform: workgroup b also clears the control words of query b
        ivf_clear_control(clr.scan_ws + (size_t)blockIdx.x * clr.ws_stride, clr.counts_off, clr.W, clr.countsA_off);
    }
    // (the workgroup's cells and those before them in the first one's row go through LDS: from memory, one after the other,
    // 64 cells took 7.4 us)
    __shared__ int32_t near[256 + IVF_MAX_NPROBE];
    const int64_t b0 = (int64_t)blockIdx.x * 256, i = b0 + threadIdx.x;
    const int64_t from = b0 / nprobe * nprobe, upto = min(b0 + 256, total);
    for (int64_t o = from + threadIdx.x; o < upto; o += 256) near[o - from] = in[o];
    __syncthreads();
    if (i >= total) return;
    const int64_t row = i / nprobe * nprobe;
    int cell = near[i - from];
    if (cell < 0 || cell >= K) cell = -1;
    bool seen = false;
#pragma unroll 8
    for (int o = (int)(row - from); o < (int)(i - from); ++o) seen |= near[o] == cell;
    if (seen) cell = -1;
    probes[i] = cell;
}

// ------------------------------------------------------------------- host

int quantize_luts(int, const float *, int, int, int, const uint8_t *, int64_t, const float *, int, int,
                  int, uint8_t *, float *, float *, float *, hipStream_t);

// Which form of ivf_tables_kernel: the sub-vector length, or 0 with the float tables by a kernel of their own before it, a
// workgroup per four (or one) probed cells -- for lengths without a form, and where one workgroup per query is too long a chain.
// That one is as long as probed cells x components; below, the float tables' way through memory costs more.  us per call,
// form of the length / 0, over 2e6 codes: 33 queries, 64 probed cells x 256 components, m = 32 104 / 105, 128 x 256 141 / 126,
// 256 x 512, m = 64 379 / 278, 256 x 1024 572 / 330; 128 queries 256 x 1024 673 / 509, 1000 queries 200 x 1024 2015 / 1869, 200 x 512
// 1400 / 1380, 200 x 128, m = 32 551 / 703, 64 x 256, m = 16 347 / 353.
static int ivf_tables_form(int d, int m, int nb, int nprobe)
{
    const int dsub = d / m;
    const int64_t chain = (int64_t)nprobe * d;
    if (dsub != 2 && dsub != 4 && dsub != 6 && dsub != 8 && dsub != 16) return 0;
    if (nb <= 128 && chain >= (dsub == 4 ? 65536 : 32768) && dsub > 2) return 0;
    return dsub == 16 && chain >= 49152 ? 0 : dsub;
}

struct IvfPlan {
    int qb, W;
    int wgs;  // workgroups a query gets of the per-query scan, at most (W: report regions laid out)
    int qd;  // queries per pass of the Index step (its distances take K floats per query)
    int seed_per_list;  // codes sampled per probed list for the bound of the scan (0: no seed kernel)
    ScanLayout l;
    size_t off_dist, off_bmin, off_front, off_probes, off_luts, off_qluts, off_qmax, off_units, off_map, off_scan, bytes;
    // shared-list scan of large batches (ivf_shared_scan): a second report region per query, the
    // pairs sorted by cell and their offsets
    bool shared;
    int shared_wgs;
    size_t stride, countsA_off, listsA_off;
    size_t off_paircnt, off_pairoff, off_item0, off_item1, off_pairs, off_taus, off_flags, off_plight, off_ulight;
    int shared_min_pairs;
};

constexpr int IVF_SHARED_PITCH = MERGE_CAP;   // keys of a query's region: what the merge kernel holds in LDS
constexpr int IVF_SHARED_MIN_Q = 384;         // smallest batch whose popular lists are scanned once for all (see shared_lists_pay)
constexpr int IVF_SHARED_MAX_R = 128;         // the region must hold a few dozen times R keys
constexpr int IVF_SHARED_MAX_K = 1 << 18;     // one workgroup sums the per-cell counts

constexpr int IVF_SHARED_MIN_PAIRS = 4;       // pairs of a cell from which its list is scanned once for all of them

int ivf_shared_scan(int, const int64_t *, const uint8_t *, int64_t, int, const int32_t *, int, int, const uint8_t *,
                    int, char *, size_t, size_t, size_t, int, unsigned *, unsigned *, unsigned *, unsigned *,
                    unsigned *, unsigned *, unsigned *, int32_t *, unsigned *, long long, int, int, hipStream_t);

// Is a batch large enough that its popular lists are scanned once for all their queries?  That costs six launches
// more (ten when the figures here were taken: some 10 to 15 us); it gains where lists are met by many queries.  From 384 queries always: what the queries meet follows from the
// lengths of the lists, which only the GPU knows, and where a few lists hold most of the codes a query-by-query scan
// reads them once per query (5e7 codes in 65536 lists of Zipf(2) lengths, 8 probes: 384 queries 12.2 against 1.7 ms,
// 4096 queries 127 against 13; Zipf(1.2), 2e7 codes, 4096 queries 9.6 against 2.5) -- while over even lists that few
// queries share it costs at most a quarter (multi-index of 1e8 codes, 512 queries 404 against 462 us; 5e7 in 65536,
// 400 queries x 64 544 against 679).  From 64 queries where an average list has 18 pairs and the queries meet
// 2.4e9 components of codes: over 2564 batches of 64 to 383 queries (16 to 2000 lists, 20 k to 8 M codes of 16 to 64
// components, even and Zipf(0.8) lengths, 7 to 48 pairs per list) the 106 that the rule takes need 0.70 of the time on
// average, the best 0.37 (8e6 codes in 16 lists, 383 queries x 2, 740 against 274 us), the worst 1.08.  Of the 1190 with 18
// pairs and fewer components 373 would be slower by 3 % and more, up to 1.6 times (2e4 codes in 64 lists, 220 queries x 6 72
// against 116: the launches alone take 35; 2.5e6 of 32 in 128, 64 x 36 191 against 260) -- over skewed lists most of them gain,
// over even ones most lose, and the host does not know the lengths.
static bool shared_lists_pay(const qadc_ivf_index *ix, int nq, int nprobe)
{
    if (nq >= IVF_SHARED_MIN_Q) return true;
    const double pairs = (double)nq * nprobe / (double)ix->K;
    return nq >= 64 && pairs >= 18.0 && pairs * (double)ix->n * (double)ix->m >= 2.4e9;
}

// small: the plan for a workspace that the best one does not fit (batches of 64 to 383 queries scan query by query).
// qadc_ivf_workspace_bytes counts both, and what this one takes is enough: see make_scan_plan.
static bool make_ivf_plan(const qadc_ivf_index *ix, int nq, int nprobe, int R, bool small, IvfPlan *p)
{
    if (!ix || nq < 1 || nprobe < 1 || nprobe > IVF_MAX_NPROBE || R < 1 || R > QADC_MAX_R) return false;
    if (!(ix->m == 8 || ix->m == 16 || ix->m == 32 || ix->m == 64)) return false;
    if (ix->d < ix->m || ix->d % ix->m || ix->K < 1 || ix->n < 0 || ix->n > 0xfffffffell) return false;
    // Most workgroups a query can get: 128 for up to 128 queries, fewer for larger calls, about
    // 16384 workgroup slots per launch (measured at N = 1e9: 4096 queries 161 K queries/s with 24 to
    // 32 against 156 K with 128; 1024 queries best with 24, 512 with 32 to 48, 256 with 64, 128 with
    // 96 to 128); the regions of a query shrink with it, so a launch holds more queries.
    // (13 to 63 queries: 256, measured 0.286 against 0.320 ms at 16 queries, 0.402 against 0.458 at 32)
    int w_def = 16384 / nq;
    if (w_def < 24) w_def = 24;
    // (up to 4 queries: 192, one query 0.0744 against 0.0780 ms)
    if (w_def > 128) w_def = (nq > IVF_WIDE_MAX_Q && nq < 64) ? 256 : nq <= 4 ? 192 : 128;
    p->W = knob_or(knobs().ivf_wgs, w_def);
    if (p->W < 1) p->W = 1;
    if (p->W > 4096) p->W = 4096;
    // Half of an average list, between 64 and 1024 codes.  With 1/16 the R-th smallest sum of the sample was so loose
    // a bound over short lists that the report lists overflowed and were cut back again and again: 1e8 codes in 16384
    // lists, 1000 queries 2.02 ms per call against 1.17, 4 queries 149 against 96 us; 4e6 in 1000, 200 queries
    // 453 against 304; 1e9 codes in 65536 lists (1024 codes against 953) the same.
    int64_t spl = ix->n / ix->K / 2;
    if (spl < 64) spl = 64;
    if (spl > 1024) spl = 1024;
    p->seed_per_list = knob_or(knobs().ivf_seed, 1) ? (int)spl : 0;
    // large batches over a moderate number of cells: every list is scanned once for all the queries
    // that probe it (QADC_IVF_SHARED=1 / 0 forces / forbids it)
    const int shared_knob = knobs().ivf_shared;
    p->shared = R <= IVF_SHARED_MAX_R && ix->K <= IVF_SHARED_MAX_K && p->seed_per_list > 0 && ix->m <= 64 &&
                (shared_knob >= 0 ? shared_knob != 0 : small ? nq >= IVF_SHARED_MIN_Q : shared_lists_pay(ix, nq, nprobe));
    // (the per-query kernel then only takes the rarely probed lists and queries that are redone: 150 queries over 1e6
    // codes spent 25 us on 109 workgroup slots per query, nearly all empty)
    p->wgs = p->shared && knobs().ivf_wgs < 0 ? std::min(p->W, 24) : p->W;
    p->l = scan_layout(p->W, R);
    p->shared_wgs = std::max(1, std::min(65535, knob_or(knobs().ivf_shared_wgs, 32768)));
    p->shared_min_pairs = std::max(1, knob_or(knobs().ivf_shared_min_pairs, IVF_SHARED_MIN_PAIRS));
    p->stride = p->l.stride;
    p->countsA_off = p->listsA_off = 0;
    if (p->shared) {
        p->countsA_off = p->l.stride;
        p->listsA_off = p->countsA_off + 256;
        p->stride = p->listsA_off + align_up((size_t)IVF_SHARED_PITCH * sizeof(uint64_t), 256);
    }
    const size_t kdist = ix->coarse ? (size_t)ix->K : 0;  // the Index step's distances
    const size_t per_q = align_up((size_t)nprobe * 4, 256) + align_up((size_t)nprobe * ix->m * 16 * 4, 256) +
                         align_up((size_t)nprobe * ix->m * 16, 256) + 256 + 4 + (size_t)p->W * 4 + p->stride +
                         (p->shared ? (size_t)nprobe * 8 + 12 : 0);
    // Queries per launch sequence.  The shared-list scan gains with every query that joins the batch
    // (more pairs per list), so it takes up to IVF_MAP_MAXQ queries in up to 1.5 GiB; the per-query
    // scan is indifferent and stays within 512 MiB.  The Index step's distances (K floats per query)
    // are computed for at most 256 MiB of queries at a time inside a sequence.
    const size_t budget = p->shared ? (1536ull << 20) : (512ull << 20);
    const size_t dist_budget = p->shared ? (256ull << 20) : 0;
    int64_t qb = (int64_t)(budget / (per_q + (p->shared ? 0 : align_up(kdist * 4, 256))));
    if (qb < 1) qb = 1;
    if (qb > nq) qb = nq;
    if (qb > IVF_MAP_MAXQ) qb = IVF_MAP_MAXQ;
    p->qb = (int)qb;
    int64_t qd = qb;  // queries per pass of the Index step
    if (dist_budget && kdist) qd = std::max<int64_t>(1, std::min<int64_t>(qb, (int64_t)(dist_budget / (kdist * 4))));
    p->qd = (int)qd;
    size_t o = 0;
    p->off_dist = o;   o += align_up((size_t)qd * kdist * 4, 256);
    p->off_bmin = o;   o += align_up((size_t)qd * ceil_div((int64_t)kdist, (int64_t)IVF_CT) * 4, 256);  // minima of the runs of cells
    // calls of up to 32 queries (ivf_front_kernel): biases [32][64], deltas, lengths of the walks, the sums of the init
    // codes [32][QADC_MAX_INIT], the minima of the tables [32][nprobe][m]
    p->off_front = o;
    o += 32 * 64 * 4 + 256 + 256 + (size_t)32 * QADC_MAX_INIT * 4 + align_up((size_t)32 * nprobe * ix->m * 4, 256);
    p->off_probes = o; o += align_up((size_t)qb * nprobe * 4, 256);
    p->off_luts = o;   o += align_up((size_t)qb * nprobe * ix->m * 16 * 4, 256);
    p->off_qluts = o;  o += align_up((size_t)qb * nprobe * ix->m * 16, 256);
    p->off_qmax = o;   o += align_up((size_t)qb * 4, 256);
    p->off_units = o;  o += align_up((size_t)qb * 4, 256);
    p->off_map = o;    o += align_up((size_t)qb * p->W * 4, 256);
    p->off_scan = o;   o += p->stride * (size_t)qb;
    p->off_paircnt = p->off_pairoff = p->off_item0 = p->off_item1 = p->off_pairs = p->off_taus = p->off_flags = 0;
    p->off_plight = p->off_ulight = 0;
    if (p->shared) {
        const size_t kk = align_up(((size_t)ix->K + 1) * 4, 256);
        p->off_paircnt = o; o += kk + 4096;  // (+ the totals of the 1024-cell blocks of the running sums)
        p->off_pairoff = o; o += kk;
        p->off_item0 = o;   o += kk;
        p->off_item1 = o;   o += kk;
        p->off_pairs = o;   o += align_up((size_t)qb * nprobe * 4, 256);
        p->off_taus = o;    o += align_up((size_t)qb * 4, 256);
        p->off_flags = o;   o += align_up((size_t)qb * 4, 256);
        p->off_plight = o;  o += align_up((size_t)qb * nprobe * 4, 256);
        p->off_ulight = o;  o += align_up((size_t)qb * 4, 256);
    }
    p->bytes = o;
    return true;
}

size_t ivf_workspace_bytes(const qadc_ivf_index *ix, int nq, int nprobe, int R)
{
    IvfPlan p, small;
    if (!make_ivf_plan(ix, nq, nprobe, R, false, &p) || !make_ivf_plan(ix, nq, nprobe, R, true, &small)) return 0;
    return std::max(p.bytes, small.bytes);
}

int ivf_search(const qadc_ivf_index *ix, const float *queries, int nq, int nprobe, int R, int init,
               int nbins, int qmin_mode, const int32_t *probes_in, uint32_t *out_ids,
               uint8_t *out_dist, int32_t *dbg_probes, uint8_t *dbg_qluts, void *workspace,
               size_t workspace_bytes, hipStream_t st)
{
    IvfPlan p, small;
    if (nq == 0) return QADC_OK;  // nothing asked for, whatever the pointers
    if (!ix || !queries || !out_ids || !out_dist)
        return fail(QADC_EINVAL, "qadc_ivf_search: null pointer");
    if (!make_ivf_plan(ix, nq, nprobe, R, false, &p) || !make_ivf_plan(ix, nq, nprobe, R, true, &small))
        return fail(QADC_EINVAL, "qadc_ivf_search: unsupported nq=%d nprobe=%d R=%d d=%d m=%d K=%d", nq,
                    nprobe, R, ix->d, ix->m, ix->K);
    if (!ix->list_off || !ix->codes || !ix->ids || !ix->codebooks)
        return fail(QADC_EINVAL, "qadc_ivf_search: index has a null pointer");
    if (!ix->coarse) {
        if (!ix->halves || !ix->cell_ids || ix->Kh < 1 || ix->Kh > 16384 || (ix->d & 1))
            return fail(QADC_EINVAL, "qadc_ivf_search: index has neither coarse centroids nor half-centroids with "
                                     "cell ids (Kh=%d d=%d)", ix->Kh, ix->d);
        if (!probes_in)
            return fail(QADC_EINVAL, "qadc_ivf_search: an index without coarse centroids is searched with probes_in "
                                     "(list numbers from qadc_multi_index_slots)");
    }
    if (init < 1 || init > QADC_MAX_INIT || nbins < 1 || nbins > 255)
        return fail(QADC_EINVAL, "qadc_ivf_search: init=%d nbins=%d", init, nbins);
    if (((uintptr_t)ix->codes & 15) != 0)
        return fail(QADC_EINVAL, "qadc_ivf_search: codes must be 16-byte aligned");
    if (!workspace || workspace_bytes < small.bytes)
        return fail(QADC_ENOMEM, "qadc_ivf_search: workspace %zu < %zu bytes", workspace_bytes, small.bytes);
    if (workspace_bytes < p.bytes) p = small;
    if (((uintptr_t)workspace & 255) != 0)
        return fail(QADC_EINVAL, "qadc_ivf_search: workspace must be 256-byte aligned");
    const int d = ix->d, m = ix->m, K = ix->K;
    char *ws = (char *)workspace;
    float *dist = (float *)(ws + p.off_dist);
    int32_t *probes = (int32_t *)(ws + p.off_probes);
    float *luts = (float *)(ws + p.off_luts);
    uint8_t *qluts = (uint8_t *)(ws + p.off_qluts);
    float *qmax = (float *)(ws + p.off_qmax);
    unsigned *qunits = (unsigned *)(ws + p.off_units);
    unsigned *wgmap = (unsigned *)(ws + p.off_map);
    char *scan_ws = ws + p.off_scan;
    const int cpt = (m / 2 <= 16) ? SCAN_VEC * (16 / (m / 2)) : 1;
    const long long unit = (long long)IVF_UNIT_TILES * IVF_NT * cpt;  // codes per unit of the scan kernel

    for (int q0 = 0; q0 < nq; q0 += p.qb) {
        const int nb = min(p.qb, nq - q0);
        const float *yq = queries + (size_t)q0 * d;
        // A few queries: Tables and the sums of the qmax walk in one launch, the quantizer's parameters in a
        // second (ivf_front_kernel, ivf_finish_kernel); the tables stay float and are quantized by the kernels that read them; the Index step's kernels
        // clear the control words.
        const bool front = nb <= 32 && !p.shared;
        float *qbias = (float *)(ws + p.off_front);
        float *qdelta = qbias + 32 * 64;
        unsigned *nwalk = (unsigned *)(qdelta + 64);
        unsigned *cand = nwalk + 64;
        unsigned *tmins = cand + (size_t)32 * QADC_MAX_INIT;
        IvfClear clr = {nullptr, 0, 0, 0, 0};
        if (front) clr = IvfClear{scan_ws, p.stride, p.l.counts_off, p.countsA_off, p.W};
        // Index
        if (probes_in) {
            const int64_t np_total = (int64_t)nb * nprobe;
            launch(QADC_PROF_IVF_INDEX, ivf_take_probes_kernel,
                   dim3((unsigned)std::max<int64_t>(ceil_div(np_total, 256), front ? nb : 0)), dim3(256), 0, st,
                   probes_in + (size_t)q0 * nprobe, nprobe, K, np_total, probes, clr, nb);
        } else {
            // large calls: bounds from the matrix units first (their factors lie where calls of a few queries keep tables)
            const bool filtered = (p.qd >= 32 || p.qd >= nb) && ivf_filter_pays(K, d, nb, nprobe) &&
                                  ivf_filter_bytes(K, d, nb) <= (size_t)p.qb * nprobe * m * 16 * 4;
            if (filtered) ivf_filter_convert(ix->coarse, K, d, yq, nb, luts, st);
            const int pass = filtered && p.qd < nb ? p.qd / 32 * 32 : p.qd;
            for (int i0 = 0; i0 < nb; i0 += pass) {
                const int ni = min(pass, nb - i0);
                const float *yi = yq + (size_t)i0 * d;
                // the minima of the runs of IVF_CT cells go with the distances, and the selection reads
                // only the runs that matter (when there are enough runs)
                unsigned *bmin = nullptr;
                const int nblk = (int)ceil_div(K, IVF_CT);
                if (nblk >= 2 * nprobe && nblk <= IVF_SEL_MAXBLK) bmin = (unsigned *)(ws + p.off_bmin);
                const IvfDistRows rows = {(size_t)d, (size_t)K, 0, 0, 0};
                if (filtered) {
                    int components = 0;
                    unsigned *rest = nullptr;
                    const float2 *qstat = ivf_filter(K, d, nb, i0, ni, luts, dist, &components, &rest, st);
                    const int vec4 = d % 4 == 0 && ((uintptr_t)ix->coarse & 15) == 0;
                    launch(QADC_PROF_IVF_INDEX, ivf_select_filtered_kernel, dim3(ni), dim3(IVF_SEL_NT), 0, st, ix->coarse,
                           K, d, yi, dist, qstat, components, nprobe, probes + (size_t)i0 * nprobe, vec4, rest);
                    // the queries that the bounds could not serve (mostly none: the workgroups return at once, 5 to 9 us a pass for both)
                    launch(QADC_PROF_IVF_INDEX, ivf_coarse_dist_kernel<8, true>, dim3((unsigned)nblk, (unsigned)ceil_div(ni, 128)),
                           dim3(256), 0, st, ix->coarse, K, d, yi, ni, rows, dist, bmin, nblk, (const unsigned *)rest);
                    launch(QADC_PROF_IVF_INDEX, ivf_select_probes_kernel<true>, dim3(ni), dim3(IVF_SEL_NT), 0, st, dist, K,
                           nprobe, probes + (size_t)i0 * nprobe, (const unsigned *)bmin, nblk, clr, (const unsigned *)rest);
                    continue;
                }
                ivf_distances(ix->coarse, K, d, yi, ni, rows, 1, dist, bmin, st);
                launch(QADC_PROF_IVF_INDEX, ivf_select_probes_kernel<false>, dim3(ni), dim3(IVF_SEL_NT), 0, st, dist, K,
                       nprobe, probes + (size_t)i0 * nprobe, (const unsigned *)bmin, nblk, clr, (const unsigned *)nullptr);
            }
        }
        IvfQuantizer fq = {nullptr, nullptr, nullptr};
        int rc = QADC_OK;
        if (front) {
            launch(QADC_PROF_IVF_TABLES, ivf_front_kernel, dim3(nprobe, nb), dim3(IVF_FRONT_NT),
                   (size_t)d * sizeof(double), st, ix->codebooks, d, m, yq, ix->coarse, ix->halves, ix->cell_ids,
                   ix->Kh, probes, nprobe, luts, ix->list_off, ix->codes, ix->n, init, unit, qunits, cand, tmins,
                   nwalk);
            launch(QADC_PROF_IVF_TABLES, ivf_finish_kernel, dim3(nb), dim3(IVF_FINISH_NT), 0, st,
                   (const unsigned *)cand, (const unsigned *)tmins, (const unsigned *)nwalk, nprobe, m, R, nbins,
                   qmin_mode, qmax, qbias, qdelta);
            fq = IvfQuantizer{luts, qbias, qdelta};
            if (dbg_qluts)  // the 8-bit tables are wanted in memory after all
                rc = quantize_luts(16, luts, nb, nprobe, m, nullptr, 0, qmax, R, nbins, qmin_mode, qluts, nullptr,
                                   nullptr, nullptr, st);
        } else {
            if (qmin_mode != QADC_QMIN_PER_TABLE && qmin_mode != QADC_QMIN_GLOBAL)
                return fail(QADC_EINVAL, "qadc_ivf_search: qmin_mode=%d", qmin_mode);
            // (a compute unit holds one workgroup of 1024 threads or two of 512: 300 queries x 64 cells 66 against 54 us)
            const int nt = m == 64 || nb <= 256 ? 1024 : 512;
#define QADC_TABLES_CASE(D_)                                                                                             \
    launch(QADC_PROF_IVF_TABLES, ivf_tables_kernel<D_>, dim3(nb), dim3(nt), 0, st, ix->codebooks, d, m, yq, ix->coarse,  \
           ix->halves, ix->cell_ids, ix->Kh, (const int32_t *)probes, nprobe, (const float *)luts, ix->list_off, ix->codes, ix->n, init, R,   \
           nbins, qmin_mode, unit, qunits, qluts, scan_ws, p.stride, p.l.counts_off, p.W, p.countsA_off,                 \
           p.shared ? (unsigned *)(ws + p.off_paircnt) : (unsigned *)nullptr, K)
            switch (ivf_tables_form(d, m, nb, nprobe)) {
            case 2: QADC_TABLES_CASE(2); break;
            case 4: QADC_TABLES_CASE(4); break;
            case 6: QADC_TABLES_CASE(6); break;
            case 8: QADC_TABLES_CASE(8); break;
            case 16: QADC_TABLES_CASE(16); break;
            default: {
                const size_t cell_bytes = (size_t)(d + m) * sizeof(double);
                const int cells = cell_bytes > 65536 ? 0 : 4 * cell_bytes > 65536 || (int64_t)nb * nprobe < 4096 ? 1 : 4;
#define QADC_FLOAT_CASE(CELLS_)                                                                                           \
    launch(QADC_PROF_IVF_TABLES, ivf_float_tables_kernel<CELLS_>,                                                        \
           dim3((unsigned)ceil_div(nprobe, std::max(1, CELLS_)), (unsigned)nb), dim3(256), CELLS_ * cell_bytes, st,       \
           ix->codebooks, d, m, yq, ix->coarse, ix->halves, ix->cell_ids, ix->Kh, (const int32_t *)probes, nprobe, luts)
                if (cells == 0) QADC_FLOAT_CASE(0);
                else if (cells == 1) QADC_FLOAT_CASE(1);
                else QADC_FLOAT_CASE(4);
#undef QADC_FLOAT_CASE
                QADC_TABLES_CASE(0);
            }
            }
#undef QADC_TABLES_CASE
        }
        if (rc != QADC_OK) return rc;
        // Scan: up to p.wgs workgroups per query, one per `upw` units of its lists (batches that fill
        // the GPU by their number alone), one per unit otherwise
        dim3 grid((unsigned)p.wgs * (unsigned)nb);
        const int upw = nb >= 64 ? min(IVF_MAX_UNITS, max(1, knob_or(knobs().ivf_units, 16))) : 1;
        // a few queries: their lists are sampled by several workgroups each
        const int seed_parts_env = knob_or(knobs().ivf_seed_parts, 0);
        // (measured at N = 1e9: one query best with 16, 16 and 32 queries with 8, 64 with 4; the shared-list
        // scan reads the bound itself and needs it in one piece)
        const int parts_def = p.shared || nb >= 256 ? 1 : nb >= 64 ? 4 : nb >= 16 ? 8 : 16;
        const int seed_parts = p.shared ? 1 : min(seed_parts_env > 0 ? seed_parts_env : parts_def, nprobe);
        // the bound is sampled from the lists of the closest cells only: they hold most of a query's best
        // codes, and the sample is most of the seed kernel's cost
        const int nseed = std::min(nprobe, std::max(1, knob_or(knobs().ivf_seed_probes, IVF_SEED_PROBES)));
        // The init codes that the sample holds (see the seed kernel).  Not where a workgroup takes longer for them than the scan of
        // the query's lists saves: fewer than 64 queries with 64-byte components (1 query of 2e7 codes, 8000 init codes 104 without,
        // 110 us per call with them; m = 32 104 / 90), and lists of a few dozen codes, nearly all sampled anyway, unless R is a small
        // part of the init codes (1e6 codes in 30000 lists, R = 100, 16 queries, 200 init codes 67 / 77, 3000 93 / 74; 70 queries, m = 8
        // 99 / 113, 1000 init codes 3 % less with them).
        const int walked = p.shared || ((nb >= 64 || m <= 32) && (p.seed_per_list > 64 || init >= 8 * R)) ? init : 0;
        unsigned *flags = p.shared ? (unsigned *)(ws + p.off_flags) : nullptr;
        IvfPairs pairs = {nullptr, nullptr, nullptr, 0};
        if (p.shared) pairs = IvfPairs{(unsigned *)(ws + p.off_paircnt), (unsigned *)(ws + p.off_taus), flags, K};
#define QADC_IVF_SEED_CASE(B_)                                                                          \
    case B_:                                                                                           \
        launch(QADC_PROF_SEED, ivf_seed_kernel<B_>, dim3(nb, seed_parts), dim3(IVF_SEED_NT), 0, st,    \
               ix->list_off, ix->codes, probes, nprobe, qluts, nbins, R, p.seed_per_list, scan_ws,     \
               p.stride, ix->n, p.shared ? 8 : 0, nseed, walked, fq, pairs);                           \
        break;
        if (p.seed_per_list > 0) {
            switch (m / 2) {
                QADC_IVF_SEED_CASE(4)
                QADC_IVF_SEED_CASE(8)
                QADC_IVF_SEED_CASE(16)
                QADC_IVF_SEED_CASE(32)
            }
        }
#undef QADC_IVF_SEED_CASE
        int32_t *probes_light = p.shared ? (int32_t *)(ws + p.off_plight) : nullptr;
        unsigned *qunits_light = p.shared ? (unsigned *)(ws + p.off_ulight) : nullptr;
        if (p.shared) {
            // the lists wanted by many queries once for all of them; then the per-query kernel takes the
            // remaining cells of every query (all cells of a query left flagged 1)
            rc = ivf_shared_scan(m / 2, ix->list_off, ix->codes, ix->n, K, probes, nb, nprobe, qluts, R, scan_ws,
                                 p.stride, p.countsA_off, p.listsA_off, IVF_SHARED_PITCH,
                                 (unsigned *)(ws + p.off_paircnt), (unsigned *)(ws + p.off_pairoff),
                                 (unsigned *)(ws + p.off_item0), (unsigned *)(ws + p.off_item1),
                                 (unsigned *)(ws + p.off_pairs), (unsigned *)(ws + p.off_taus), flags, probes_light,
                                 qunits_light, unit, p.shared_min_pairs, p.shared_wgs, st);
            if (rc != QADC_OK) return rc;
        }
        // (a few queries need no map: every query gets its p.wgs workgroup slots in turn)
        const bool mapped = nb >= 64 || p.shared;
        // a few queries: workgroups of 1024 threads (measured at N = 1e9: 1 query 0.121 against 0.136 ms,
        // 4 queries 0.163 against 0.181, 8 queries 0.208 against 0.220, 12 the same, 16 slower)
        const bool wide_wgs = !mapped && nb <= knob_or(knobs().ivf_wide_q, IVF_WIDE_MAX_Q);
        if (mapped)
            launch(QADC_PROF_SEED, ivf_wgmap_kernel, dim3(16), dim3(IVF_MAP_NT), 0, st, qunits, nb, upw, p.wgs, wgmap,
                   (const unsigned *)qunits_light, (const unsigned *)flags);
        const int hist_bound = (p.seed_per_list > 0 && seed_parts > 1) ? 1 : 0;
#define QADC_IVF_CASE(B_)                                                                              \
    case B_:                                                                                          \
        if (wide_wgs)                                                                                  \
            launch(QADC_PROF_SCAN, ivf_scan_kernel<B_, 1024>, grid, dim3(1024), 0, st, ix->list_off, ix->codes, \
                   ix->n, probes, nprobe, qluts, nbins, R, upw, p.wgs, mapped ? wgmap : (unsigned *)nullptr, scan_ws, \
                   p.stride, p.l.counts_off, p.l.lists_off, (const int32_t *)probes_light,              \
                   (const unsigned *)flags, fq, hist_bound);                                           \
        else                                                                                           \
            launch(QADC_PROF_SCAN, ivf_scan_kernel<B_, IVF_NT>, grid, dim3(IVF_NT), 0, st, ix->list_off, ix->codes, \
                   ix->n, probes, nprobe, qluts, nbins, R, upw, p.wgs, mapped ? wgmap : (unsigned *)nullptr, scan_ws, \
                   p.stride, p.l.counts_off, p.l.lists_off, (const int32_t *)probes_light,              \
                   (const unsigned *)flags, fq, hist_bound);                                           \
        break;
        switch (m / 2) {
            QADC_IVF_CASE(4)
            QADC_IVF_CASE(8)
            QADC_IVF_CASE(16)
            QADC_IVF_CASE(32)
        }
#undef QADC_IVF_CASE
        uint32_t *oi = out_ids + (size_t)q0 * R;
        rc = launch_merge<uint8_t, 5>(nb, st, front ? MERGE_FILLED : MERGE_MIXED, scan_ws, p.stride, p.l.counts_off, p.l.lists_off, p.wgs,
                                      (unsigned)R, R, (uint8_t)nbins, oi, out_dist + (size_t)q0 * R, p.countsA_off,
                                      p.listsA_off, p.shared ? 1 : 0, p.shared ? IVF_SHARED_PITCH : 0, flags,
                                      (const uint32_t *)ix->ids, (int64_t)ix->n);  // positions -> vector ids
        if (rc != QADC_OK) return rc;
        if (dbg_probes)
            QADC_HIP_TRY(hipMemcpyAsync(dbg_probes + (size_t)q0 * nprobe, probes,
                                        (size_t)nb * nprobe * sizeof(int32_t), hipMemcpyDeviceToDevice, st));
        if (dbg_qluts)
            QADC_HIP_TRY(hipMemcpyAsync(dbg_qluts + (size_t)q0 * nprobe * m * 16, qluts,
                                        (size_t)nb * nprobe * m * 16, hipMemcpyDeviceToDevice, st));
    }
    QADC_HIP_TRY(hipGetLastError());
    return QADC_OK;
}

}  // namespace qadc
