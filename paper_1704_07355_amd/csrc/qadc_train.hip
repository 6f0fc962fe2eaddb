// Product-quantizer training on gfx950 (Section 2.1 of the paper: one k-centroid codebook
// per sub-space, each a Lloyd k-means).  Database side, not on the query path: it exists so
// that large synthetic databases can be trained, encoded and searched without leaving HBM.
//
// One iteration = assign every learning vector's sub-vector to its closest centroid
// (float64 distances from the differences, ties to the lowest index), then replace each
// centroid by the mean of its sub-vectors (float64 sum in row order, stored as float32);
// a centroid that owns nothing keeps its value.  No atomics: the result is deterministic.

#include <type_traits>

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

// Means of the sub-vectors of one centroid: workgroup (i, j, block of TRAIN_TD dimensions).  The mean is defined by the
// float64 sum in row order, one chain of additions per component; a chain per component is what this kernel was bound by
// (44 us per iteration for 20,000 rows, m = 16, 16 centroids, 8 dimensions).  The sum is taken in many chains instead, a
// lane per (row slot, component), together with the sum of the absolute values: `cnt` additions in a row are off by at
// most cnt 2^-53 times that, these by what the longest of their chains adds (the first slot's, counted round by round: a
// round of few rows leaves most slots without one), and unless the float32 rounding of the mean changes within this margin
// it is the row-order one.  Where it does (about one mean in 10^5 of a thousand rows), or is not a
// number, the workgroup walks its rows again in row order.
// The labels, a column of the label matrix, are read in rounds, and the numbers of the centroid's rows are left in LDS in
// row order (bits of the labels that match, ballots of the lanes' counts; no atomics).  Bound by the instructions of that search
// and by round trips: labels, then rows four to twelve loads at a time, as many as the longest slot has.  (A label a lane
// and instruction, eight loads in flight and halves of the sums' tree: 20,000 rows, m = 16, 16 centroids of 8 dimensions, 17.1
// us per iteration with the assignment, now 16.4; 20,000, 256 of 8 104 -> 97; 300,001, 256 of 16 1805 -> 1488; 1 M, 16 of 8 502 -> 469.)
// 44 -> 11.6 us per iteration where no mean is in doubt; 1 M rows, where one iteration in three has one, 2.4 -> 0.5 ms per
// iteration with the assignment; learning sets of NaN, all rows in order, a tenth slower than before, and 4 to 9 % where most
// workgroups have one of their 64 means in doubt (300,000 to 600,000 rows, 16 centroids near zero, 120 components and more).
constexpr int TRAIN_TD = 64;                             // components per workgroup, at most
constexpr unsigned TRAIN_FEW = 128;                      // rows that are added in order right away
constexpr int TRAIN_STAGE = 4096;                        // components fetched at a time for the sum in row order

// Leaves the numbers (relative to `base`) of the rows base .. base + NT * PER - 1 with label i in `rows`, in row order;
// returns how many.  Every thread of the workgroup calls it; ends with a barrier.
template <int NT, int PER>
__device__ __forceinline__ unsigned train_rows(const uint8_t *__restrict__ col, int64_t base, int64_t n, unsigned i,
                                               uint16_t *rows, unsigned *wcount, unsigned *fetched)
{
    static_assert(PER % 4 == 0 && PER < 32, "whole words, and counts of five bits");
    const int lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x / WAVE;
    // a wavefront fetches 64 PER labels, 256 at a time, and a lane looks at PER in a row: bit k of `own` is set where number k is i
    constexpr int WORDS = PER / 4;
    const unsigned at0 = threadIdx.x * PER;
    const int64_t first = base + wave * (WAVE * PER);
    unsigned *mine_in = fetched + wave * (WAVE * WORDS);
    unsigned w[WORDS];
#pragma unroll
    for (int k = 0; k < WORDS; ++k) {
        const int64_t at = first + (k * WAVE + lane) * 4;
        w[k] = (i ^ 1u) * 0x01010101u;  // (a label that is not there is one that is not i)
        if (at + 4 <= n) __builtin_memcpy(&w[k], col + at, 4);
    }
    if (first + WAVE * PER > n) {  // uniform: the last word may be a part of one
#pragma unroll
        for (int k = 0; k < WORDS; ++k)
            for (int u = 0; u < 3; ++u) {
                const int64_t at = first + (k * WAVE + lane) * 4;
                if (at + 4 > n && at + u < n) w[k] = (w[k] & ~(255u << (8 * u))) | (unsigned)col[at + u] << (8 * u);
            }
    }
#pragma unroll
    for (int k = 0; k < WORDS; ++k) mine_in[k * WAVE + lane] = w[k];
    __builtin_amdgcn_wave_barrier();  // (a wavefront's LDS accesses are in order; the compiler keeps them so)
    unsigned own = 0;
#pragma unroll
    for (int k = 0; k < WORDS; ++k) {
        const unsigned x = mine_in[lane * WORDS + k] ^ i * 0x01010101u;
        const unsigned zero = ~(((x & 0x7f7f7f7fu) + 0x7f7f7f7fu) | x | 0x7f7f7f7fu);  // bit 7 of a byte: it was i
        own |= ((zero >> 7) * 0x10204080u >> 28) << (4 * k);
    }
    const unsigned mine = (unsigned)__popc(own);
    unsigned before = 0, total = 0;  // rows of the lanes before this one, of the wavefront
#pragma unroll
    for (int b = 0; b < 5; ++b) {
        const unsigned long long mask = __ballot(mine >> b & 1u);
        before += rank_in_mask(mask) << b;
        total += (unsigned)__popcll(mask) << b;
    }
    if (lane == 0) wcount[wave] = total;
    __syncthreads();
    unsigned at = before, found = 0;
#pragma unroll
    for (int w = 0; w < NT / WAVE; ++w) {
        const unsigned c = wcount[w];
        if (w < wave) at += c;
        found += c;
    }
    for (unsigned left = own; left != 0; left &= left - 1) rows[at++] = (uint16_t)(at0 + (unsigned)__ffs((int)left) - 1);
    __syncthreads();
    return found;
}

// NT threads, PER labels per lane and round.
template <int NT, int PER>
__global__ __launch_bounds__(NT) void train_update_kernel(
    const float *__restrict__ train, int64_t n, int d, int m, int ksub, const uint8_t *__restrict__ labels,
    float *__restrict__ cb)
{
    constexpr int SEG = NT * PER;                        // labels per round
    __shared__ uint16_t rows[SEG];                 // the centroid's rows of the round, in row order
    __shared__ union {
        double2 part[NT];                          // (sum, sum of absolute values) of a slot and component
        float stage[2][TRAIN_STAGE];
        unsigned labels[SEG / 4];                  // of the round, while its rows are looked for
    } sh;
    __shared__ unsigned wcount[NT / WAVE];
    double2 *part = sh.part;
    const int tid = threadIdx.x;
    const int dsub = d / m;
    // workgroups that read neighbouring components are on one XCD, whose L2 then holds what they share of a row's lines
    const unsigned xcd = gridDim.x / 8, wg = xcd * 8 == gridDim.x ? (blockIdx.x % 8) * xcd + blockIdx.x / 8 : blockIdx.x;
    const int i = (int)(wg % (unsigned)ksub), jt = (int)(wg / (unsigned)ksub);
    const int blocks_t = (dsub + TRAIN_TD - 1) / TRAIN_TD;
    const int j = jt / blocks_t, t0 = (jt - j * blocks_t) * TRAIN_TD;
    const int td = min(TRAIN_TD, dsub - t0);
    const uint8_t *col = labels + (size_t)j * n;
    const float *src = train + (size_t)j * dsub + t0;
    float *out = cb + ((size_t)j * ksub + i) * dsub + t0;
    double sum = 0.0;
    int64_t cnt = 0;
    if (n > SEG || (cnt = train_rows<NT, PER>(col, 0, n, (unsigned)i, rows, wcount, sh.labels)) > TRAIN_FEW) {  // uniform
        double mag = 0.0;
        int64_t chain = 0;                         // additions of this slot (the first, with the most, decides below)
        const int slots = NT / td;                 // rows side by side
        const int slot = tid / td, t = tid - slot * td;
        for (int64_t base = 0; base < n; base += SEG) {
            const unsigned found = n <= SEG ? (unsigned)cnt : train_rows<NT, PER>(col, base, n, (unsigned)i, rows, wcount, sh.labels);
            if (n > SEG) cnt += found;
            if (slot < slots) {
                const float *from = src + base * d + t;
                // U of the slot's rows from row r0 on, their loads in flight together
                auto add = [&](auto many, unsigned r0) {
                    constexpr int U = decltype(many)::value;
                    float v[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) v[u] = from[(int64_t)rows[min(r0 + u * (unsigned)slots, found - 1)] * d];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const double x = (double)(r0 + u * (unsigned)slots < found ? v[u] : 0.0f);
                        sum += x;
                        mag += fabs(x);
                    }
                    chain += U;
                };
                const unsigned most = (found + (unsigned)slots - 1) / (unsigned)slots;  // a slot's rows
                unsigned r = 0;
                for (; r + 8 < most; r += 12) add(std::integral_constant<int, 12>(), slot + r * slots);
                if (r + 4 < most) add(std::integral_constant<int, 8>(), slot + r * slots);
                else if (r < most) add(std::integral_constant<int, 4>(), slot + r * slots);
            }
            __syncthreads();                             // `rows` and `wcount` are written again in the next round
        }
        int parts = slots;
        if (td < WAVE && (td & (td - 1)) == 0) {         // uniform: the lanes of a wavefront that hold a component, by shuffles
            for (int k = td; k < WAVE; k *= 2) {
                sum += __shfl_xor(sum, k);
                mag += __shfl_xor(mag, k);
            }
            parts = NT / WAVE;
            if ((tid & (WAVE - 1)) < td) part[tid / WAVE * td + t] = make_double2(sum, mag);
        } else {
            part[tid] = make_double2(sum, mag);
        }
        __syncthreads();
        // an eighth of the slots, then an eighth of those
        for (int have = parts; have > 1;) {              // uniform
            const int next = (have + 7) / 8;
            if (slot < next) {
                double2 all = part[tid];
#pragma unroll
                for (int u = 1; u < 8; ++u) {
                    const double2 o = part[min(slot + u * next, have - 1) * td + t];
                    if (slot + u * next < have) all = make_double2(all.x + o.x, all.y + o.y);
                }
                part[tid] = all;
            }
            __syncthreads();
            have = next;
        }
        bool sure = true;
        float mean = 0.0f;
        if (tid < td) {
            const double s = part[tid].x, c = (double)cnt;
            // row order: cnt additions; here: those of the longest chain and at most 21 of the tree (NT / td slots, or 6 and
            // 14 of the shuffles' 16).  (1.01: the rounding of
            // this line and of the two divisions below is far under a hundredth of it)
            const double eps = part[tid].y * (c + (double)chain + 28.0) * (1.01 * 0x1p-53);
            mean = (float)(s / c);
            sure = __float_as_uint((float)((s - eps) / c)) == __float_as_uint((float)((s + eps) / c)) &&
                   __builtin_isfinite(mean);
        }
        if (cnt == 0) return;                            // uniform
        if (!__syncthreads_or(!sure)) {                  // uniform; (a barrier: the parts have been read)
            if (tid < td) out[tid] = mean;
            return;
        }
        sum = 0.0;
    }
    // The definition: a stage of rows is fetched by all while the one before is added in order, a thread per component.
    const int per_stage = TRAIN_STAGE / td;              // rows
    for (int64_t base = 0; base < n; base += SEG) {
        const int found = n <= SEG ? (int)cnt      // `rows` still holds them
                                         : (int)train_rows<NT, PER>(col, base, n, (unsigned)i, rows, wcount, sh.labels);
        const int stages = (found + per_stage - 1) / per_stage;
        for (int s = 0; s <= stages; ++s) {              // uniform
            if (s < stages) {
                const int r0 = s * per_stage, elems = min(per_stage, found - r0) * td;
                for (int e0 = tid; e0 < elems; e0 += 4 * NT) {
                    float v[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int e = min(e0 + u * NT, elems - 1), r = e / td;
                        v[u] = src[(base + rows[r0 + r]) * d + (e - r * td)];
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (e0 + u * NT < elems) sh.stage[s & 1][e0 + u * NT] = v[u];
                }
            }
            if (s > 0 && tid < td) {
                const float *from = sh.stage[(s - 1) & 1] + tid;
                const int have = min(per_stage, found - (s - 1) * per_stage);
                int r = 0;
                for (; r + 16 <= have; r += 16) {
                    float v[16];
#pragma unroll
                    for (int u = 0; u < 16; ++u) v[u] = from[(r + u) * td];
#pragma unroll
                    for (int u = 0; u < 16; ++u) sum += (double)v[u];
                }
                for (; r < have; ++r) sum += (double)from[r * td];
            }
            __syncthreads();
        }
    }
    if (cnt > 0 && tid < td) out[tid] = (float)(sum / (double)cnt);
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
        const dim3 grid((unsigned)(ksub * m * ceil_div(d / m, TRAIN_TD)));
        // (a few hundred rows: the launch counts, 11.9 us per iteration with 1024 threads, 11.2 with 512; 20,000 rows 19 and 22.
        // Five iterations with the assignment, 1024 threads / 512: 5000 rows m = 8, 256 centroids of 12 components 592 / 455 us,
        // m = 16, 16 of 8 69 / 58; 8192 rows m = 8, 16 centroids of 120 588 / 614, 256 of 12 607 / 459: the rows of one round of
        // 512 x 16 labels, and as many workgroups as fit, where few rows are a centroid's)
        if (n <= 4096)
            hipLaunchKernelGGL((train_update_kernel<512, 8>), grid, dim3(512), 0, st, train, n, d, m, ksub, labels,
                               codebooks);
        else if (n <= 8192)
            hipLaunchKernelGGL((train_update_kernel<512, 16>), grid, dim3(512), 0, st, train, n, d, m, ksub, labels,
                               codebooks);
        else
            hipLaunchKernelGGL((train_update_kernel<1024, 20>), grid, dim3(1024), 0, st, train, n, d, m, ksub, labels,
                               codebooks);
    }
    QADC_HIP_TRY(hipGetLastError());
    return QADC_OK;
}

}  // namespace qadc
