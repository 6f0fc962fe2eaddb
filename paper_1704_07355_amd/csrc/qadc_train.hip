// Product-quantizer training on gfx950 (Section 2.1 of the paper: one k-centroid codebook
// per sub-space, each a Lloyd k-means).  Database side, not on the query path: it exists so
// that large synthetic databases can be trained, encoded and searched without leaving HBM.
//
// One iteration = assign every learning vector's sub-vector to its closest centroid
// (float64 distances from the differences, ties to the lowest index), then replace each
// centroid by the mean of its sub-vectors (float64 sum in row order, stored as float32);
// a centroid that owns nothing keeps its value.  No atomics: the result is deterministic.

#include "qadc_nearest.h"

namespace qadc {

// A row number outside [0, n) is clamped to the nearest row: nothing outside `train` is read.
__global__ void train_init_kernel(const float *__restrict__ train, int64_t n, int d, int m, int ksub,
                                  const int64_t *__restrict__ init_rows, float *__restrict__ cb)
{
    const int dsub = d / m;
    const int e = blockIdx.x * blockDim.x + threadIdx.x;  // (j, i, t)
    if (e >= m * ksub * dsub) return;
    const int t = e % dsub, i = (e / dsub) % ksub, j = e / (dsub * ksub);
    const int64_t row = min(max(init_rows[i], (int64_t)0), n - 1);
    cb[e] = train[row * d + j * dsub + t];
}

// labels[j][r] = closest centroid of sub-vector j of row r.  A wavefront takes 64 rows and one sub-quantizer
// (qadc_nearest.h); the labels are stored a column per sub-quantizer, as the update reads them.  20,000 rows of
// 128 dimensions, m = 16, 16 centroids: 145 -> 6 us.
template <int KSUB, int DS>
__global__ __launch_bounds__(256) void train_assign_kernel(const float *__restrict__ train, int64_t n, int d, int m,
                                                           const float *__restrict__ cb, uint8_t *__restrict__ labels)
{
    const int dsub = DS ? DS : d / m;
    const int64_t unit = (int64_t)blockIdx.x * (256 / WAVE) + __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const int64_t block = unit / m;
    const int j = (int)(unit - block * m);
    if (block * WAVE >= n) return;  // uniform
    const int64_t r = block * WAVE + (threadIdx.x & (WAVE - 1));
    const float *xs = train + min(r, n - 1) * d + (int64_t)j * dsub;
    float xv[DS ? DS : 1];
    if constexpr (DS != 0) {
#pragma unroll
        for (int t = 0; t < DS; ++t) xv[t] = xs[t];
    }
    const unsigned a = nearest_centroid<KSUB, DS>(xv, xs, nullptr, cb + (size_t)j * KSUB * dsub, dsub, r < n);
    if (r < n) labels[(size_t)j * n + r] = (uint8_t)a;
}

template <int KSUB>
static void launch_train_assign(const float *train, int64_t n, int d, int m, const float *cb, uint8_t *labels,
                                hipStream_t st)
{
    const dim3 grid((unsigned)ceil_div(ceil_div(n, WAVE) * m, 256 / WAVE));
#define QADC_ASG(D_)                                                                                          \
    case D_:                                                                                                  \
        hipLaunchKernelGGL((train_assign_kernel<KSUB, D_>), grid, dim3(256), 0, st, train, n, d, m, cb, labels); \
        return;
    switch (d / m) {
    QADC_ASG(2) QADC_ASG(3) QADC_ASG(4) QADC_ASG(6) QADC_ASG(8) QADC_ASG(12) QADC_ASG(16)
    default:
        hipLaunchKernelGGL((train_assign_kernel<KSUB, 0>), grid, dim3(256), 0, st, train, n, d, m, cb, labels);
    }
#undef QADC_ASG
}

// Means of the sub-vectors of one centroid: workgroup (i, j, block of TRAIN_TD dimensions).  The
// row-order float64 sum of a component is one chain of additions, so what a workgroup can do is keep
// everything else out of that chain: its eight wavefronts read TRAIN_SEG labels at a time, a column of
// the label matrix, and leave the numbers of the centroid's rows in LDS in row order (ballots and running
// counts, no atomics); they then fetch the rows' components a stage at a time, all loads of a stage in
// flight together, and while the next stage is fetched the first wavefront adds the stage before it, a
// lane per component, from LDS.  Bound by the chain of float64 additions over the centroid's rows.
// 20,000 rows, m = 16, 16 centroids, 8 dimensions: 4000 us (one thread per component walking all rows:
// 32 wavefronts, a dependent label load per row) -> 46 us.
constexpr int TRAIN_NT = 512;
constexpr int TRAIN_WAVES = TRAIN_NT / WAVE;
constexpr int TRAIN_PER = 16;                            // labels per lane and round
constexpr int TRAIN_SEG = TRAIN_NT * TRAIN_PER;          // labels per round
constexpr int TRAIN_TD = 64;                             // components per workgroup, at most: a lane each
constexpr int TRAIN_STAGE = 4096;                        // values per stage, already float64: the adding lane has nothing to convert

__global__ __launch_bounds__(TRAIN_NT) void train_update_kernel(
    const float *__restrict__ train, int64_t n, int d, int m, int ksub, const uint8_t *__restrict__ labels,
    float *__restrict__ cb)
{
    __shared__ uint16_t rows[TRAIN_SEG];                 // the centroid's rows of the round, in row order
    __shared__ double stage[2][TRAIN_STAGE];
    __shared__ unsigned wcount[TRAIN_WAVES];
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
    const int dsub = d / m;
    const int i = (int)(blockIdx.x % (unsigned)ksub), jt = (int)(blockIdx.x / (unsigned)ksub);
    const int blocks_t = (dsub + TRAIN_TD - 1) / TRAIN_TD;
    const int j = jt / blocks_t, t0 = (jt - j * blocks_t) * TRAIN_TD;
    const int td = min(TRAIN_TD, dsub - t0);
    const int per_stage = TRAIN_STAGE / td;              // rows per stage
    const uint8_t *col = labels + (size_t)j * n;
    const float *src = train + (size_t)j * dsub + t0;
    double sum = 0.0;
    int64_t cnt = 0;
    for (int64_t base = 0; base < n; base += TRAIN_SEG) {
        // wavefront w looks at labels base + w * 1024 + k * 64 + lane, k = 0 .. 15
        const int64_t first = base + (int64_t)wave * (WAVE * TRAIN_PER) + lane;
        unsigned lab[TRAIN_PER];
#pragma unroll
        for (int k = 0; k < TRAIN_PER; ++k) lab[k] = (first + k * WAVE < n) ? col[first + k * WAVE] : 0xffffu;
        unsigned mine = 0;
#pragma unroll
        for (int k = 0; k < TRAIN_PER; ++k) mine += (unsigned)__popcll(__ballot(lab[k] == (unsigned)i));
        if (lane == 0) wcount[wave] = mine;
        __syncthreads();
        unsigned at = 0, found = 0;
#pragma unroll
        for (int w = 0; w < TRAIN_WAVES; ++w) {
            const unsigned c = wcount[w];
            if (w < wave) at += c;
            found += c;
        }
#pragma unroll
        for (int k = 0; k < TRAIN_PER; ++k) {
            const bool own = lab[k] == (unsigned)i;
            const unsigned long long mask = __ballot(own);
            if (own) rows[at + rank_in_mask(mask)] = (uint16_t)(first + k * WAVE - base);
            at += (unsigned)__popcll(mask);
        }
        __syncthreads();
        cnt += found;
        // stage s is fetched while stage s - 1 is added
        const int stages = ((int)found + per_stage - 1) / per_stage;
        for (int s = 0; s <= stages; ++s) {              // uniform
            if (s < stages) {
                const int r0 = s * per_stage;
                const int elems = min(per_stage, (int)found - r0) * td;
                double *to = stage[s & 1];
                constexpr int FL = 8;                    // loads in flight per thread
                for (int e0 = tid; e0 < elems; e0 += FL * TRAIN_NT) {
                    float v[FL];
#pragma unroll
                    for (int u = 0; u < FL; ++u) {
                        const int e = min(e0 + u * TRAIN_NT, elems - 1);
                        const int r = e / td, t = e - r * td;
                        v[u] = src[(base + rows[r0 + r]) * d + t];
                    }
#pragma unroll
                    for (int u = 0; u < FL; ++u)
                        if (e0 + u * TRAIN_NT < elems) to[e0 + u * TRAIN_NT] = (double)v[u];
                }
            }
            if (s > 0 && tid < td) {
                const double *from = stage[(s - 1) & 1] + tid;
                const int have = min(per_stage, (int)found - (s - 1) * per_stage);
                int r = 0;
                if (have >= 16) {  // the next sixteen rows are read from LDS while sixteen are added
                    double v[16];
#pragma unroll
                    for (int u = 0; u < 16; ++u) v[u] = from[u * td];
                    for (r = 16; r + 16 <= have; r += 16) {
                        double nx[16];
#pragma unroll
                        for (int u = 0; u < 16; ++u) nx[u] = from[(r + u) * td];
#pragma unroll
                        for (int u = 0; u < 16; ++u) sum += v[u];
#pragma unroll
                        for (int u = 0; u < 16; ++u) v[u] = nx[u];
                    }
#pragma unroll
                    for (int u = 0; u < 16; ++u) sum += v[u];
                }
                for (; r < have; ++r) sum += from[r * td];
            }
            __syncthreads();
        }
    }
    if (tid < td && cnt) cb[((size_t)j * ksub + i) * dsub + t0 + tid] = (float)(sum / (double)cnt);
}

int pq_train(const float *train, int64_t n, int d, int m, int ksub, const int64_t *init_rows, int iters,
             float *codebooks, void *workspace, size_t workspace_bytes, hipStream_t st)
{
    if (!train || !init_rows || !codebooks) return fail(QADC_EINVAL, "qadc_pq_train: null pointer");
    if (m < 1 || d < m || d % m != 0 || (ksub != 16 && ksub != 64 && ksub != 256) || n < 1 || iters < 0)
        return fail(QADC_EINVAL, "qadc_pq_train: unsupported n=%lld d=%d m=%d ksub=%d iters=%d",
                    (long long)n, d, m, ksub, iters);
    if (!workspace || workspace_bytes < (size_t)n * m)
        return fail(QADC_ENOMEM, "qadc_pq_train: workspace %zu < %zu bytes", workspace_bytes, (size_t)n * m);
    uint8_t *labels = (uint8_t *)workspace;
    const int entries = m * ksub * (d / m);
    hipLaunchKernelGGL(train_init_kernel, dim3((unsigned)ceil_div(entries, 256)), dim3(256), 0, st, train,
                       n, d, m, ksub, init_rows, codebooks);
    for (int it = 0; it < iters; ++it) {
        if (ksub == 16) launch_train_assign<16>(train, n, d, m, codebooks, labels, st);
        else if (ksub == 64) launch_train_assign<64>(train, n, d, m, codebooks, labels, st);
        else launch_train_assign<256>(train, n, d, m, codebooks, labels, st);
        hipLaunchKernelGGL(train_update_kernel,
                           dim3((unsigned)(ksub * m * ceil_div(d / m, TRAIN_TD))), dim3(TRAIN_NT), 0, st, train, n, d,
                           m, ksub, labels, codebooks);
    }
    QADC_HIP_TRY(hipGetLastError());
    return QADC_OK;
}

}  // namespace qadc
