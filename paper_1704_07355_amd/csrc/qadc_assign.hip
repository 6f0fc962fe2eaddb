// Cell of a vector on gfx950 (Section 2.2 of the paper): cell(x) = index of the closest coarse centroid,
// float64 distances from the differences (one fused multiply-add per component, increasing component),
// the lowest cell among equal distances -- the vector quantizer q_i of the inverted index.
//
// assign_filter_kernel (d <= 256) finds that cell without forming all n x K float64 distances.  With x' and
// c' the differences to a reference vector, |x - c|^2 = |x'|^2 + |c'|^2 - 2 x'.c', and the part that depends
// on the cell is a matrix product: both factors are split into two bfloat16 numbers (16 significant bits)
// and hi.hi + hi.lo + lo.hi is summed in float32 by the matrix units.  A lane keeps, per vector, the three
// smallest of its group minima (a group: the 16 cells of a result tile that lie in one lane).  Whatever the
// rounding, the closest cell lies in a group whose minimum is within a margin (bound below) of the smallest;
// those groups -- mostly one -- are measured in float32 and, cells that come within its rounding of each other, in
// float64 by the definition.  A vector that may have more of them than a lane remembers (more than two equal
// centroids, values beyond the float32 range, infinities, NaN) is marked, and assign_rest_kernel measures it
// against all cells.  The result is the definition's, whatever the route.
//
// Bound: 3 x 2 n K d operations on the matrix units.  Measured for 1 M vectors, d = 128, K = 4096: 2.8 ms =
// 1.1 PFLOP/s of bfloat16 products (the float64 kernel: 37.5 ms); 2.0 ms of it are products and group minima,
// 0.4 splitting the centroids, which every workgroup does again -- so eight wavefronts share the tiles and hold
// the operands of 64 vectors each for the whole walk, all but a few of them in registers (256 per lane; 10
// spilled for d = 128; the form for d = 129 to 255 and other rows spills 46 and takes 2.5 ms for 262 k vectors, d = 200,
// K = 4096: 17.2 in float64) -- and 0.5 the last step.
// A margin is a matter of the vector and of the closest cells: a far or NaN centroid costs the other cells
// nothing (2.8 ms; with one margin for all, from the farthest centroid, 122).  Every centroid twice: 1.0 ms for 262 k
// vectors (4.5 when every cell of a group was measured in float64, a lane per row).  Every centroid four times, all
// vectors marked: 45 ms per 1 M (69 when the filter's own workgroups walked over the cells, a lane per row).
//
// assign_f64_kernel (d > 256: the vectors no longer fit the registers): a workgroup of 256 threads takes 128
// vectors and walks over all cells 128 at a time; 16 components of both go through LDS as float64 per step,
// every thread accumulates 8 x 8 distances and keeps, per vector, the best of the cells it has seen; the 16
// threads of a vector compare their candidates at the end under the order (distance, cell).  Vector-ALU
// bound: 2 float64 operations per (vector, cell, component), 54 % of the float64 vector peak.

#include "qadc_common.h"

namespace qadc {

// ------------------------------------------------------------------ float64

constexpr int ASG_TM = 128;  // vectors per workgroup
constexpr int ASG_TN = 128;  // cells per step
constexpr int ASG_TK = 16;   // components per step
constexpr int ASG_LD = ASG_TM + 2;  // row stride in doubles: keeps 16-byte alignment, shifts the banks

struct AssignTile {
    __attribute__((aligned(16))) double xs[ASG_TK][ASG_LD];
    __attribute__((aligned(16))) double cs[ASG_TK][ASG_LD];
    double cand_d[ASG_TM][16];
    int cand_c[ASG_TM][16];
};

// The cells of up to ASG_TM vectors, by a workgroup of 256 threads; row(k): the row of x that is vector k of the tile, -1
// for none.
// Thread (tx, ty), tx = tid & 15, ty = tid >> 4, owns the vectors 8*ty .. 8*ty+7 of the tile and
// the cells 32*k + 2*tx + e (k < 4, e < 2): a wavefront's 16-byte reads of the cells are
// contiguous across its lanes, its reads of the vectors are the same for 16 lanes.
template <typename Row, typename Store>
__device__ __forceinline__ void assign_tile(AssignTile &s, const float *__restrict__ coarse, int K, int d,
                                            const float *__restrict__ x, int64_t ldx, Row row, Store store)
{
    const int tid = threadIdx.x;
    const int tx = tid & 15, ty = tid >> 4;
    double best_d[8];
    int best_c[8];
    int from[8];  // the rows this thread fetches from
#pragma unroll
    for (int a = 0; a < 8; ++a) { best_d[a] = __builtin_inf(); best_c[a] = 0x7fffffff; from[a] = row(ty + 16 * a); }

    for (int c0 = 0; c0 < K; c0 += ASG_TN) {
        double acc[8][8];
#pragma unroll
        for (int a = 0; a < 8; ++a)
#pragma unroll
            for (int b = 0; b < 8; ++b) acc[a][b] = 0.0;
        for (int t0 = 0; t0 < d; t0 += ASG_TK) {
            // 128 x 16 elements of x and of the centroids, eight of each per thread, zero beyond the edges
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int idx = tid + e * 256;
                const int r = idx >> 4, col = idx & 15;
                const int t = t0 + col;
                const int c = c0 + r;
                s.xs[col][r] = (from[e] >= 0 && t < d) ? (double)x[from[e] * ldx + t] : 0.0;
                s.cs[col][r] = (c < K && t < d) ? (double)coarse[(size_t)c * d + t] : 0.0;
            }
            __syncthreads();
#pragma unroll 4
            for (int kk = 0; kk < ASG_TK; ++kk) {
                double xv[8], cv[8];
#pragma unroll
                for (int a = 0; a < 8; a += 2) {
                    const double2 v = *reinterpret_cast<const double2 *>(&s.xs[kk][8 * ty + a]);
                    xv[a] = v.x; xv[a + 1] = v.y;
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const double2 v = *reinterpret_cast<const double2 *>(&s.cs[kk][32 * k + 2 * tx]);
                    cv[2 * k] = v.x; cv[2 * k + 1] = v.y;
                }
#pragma unroll
                for (int a = 0; a < 8; ++a)
#pragma unroll
                    for (int b = 0; b < 8; ++b) {
                        const double df = xv[a] - cv[b];
                        acc[a][b] = fma(df, df, acc[a][b]);
                    }
            }
            __syncthreads();
        }
        // the smaller distance wins, the lower cell among equal distances
#pragma unroll
        for (int a = 0; a < 8; ++a)
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const int c = c0 + 32 * (b >> 1) + 2 * tx + (b & 1);
                if (c < K && (acc[a][b] < best_d[a] || (acc[a][b] == best_d[a] && c < best_c[a]))) {
                    best_d[a] = acc[a][b];
                    best_c[a] = c;
                }
            }
    }
#pragma unroll
    for (int a = 0; a < 8; ++a) {
        s.cand_d[8 * ty + a][tx] = best_d[a];
        s.cand_c[8 * ty + a][tx] = best_c[a];
    }
    __syncthreads();
    if (tid < ASG_TM && row(tid) >= 0) {
        double bd = s.cand_d[tid][0];
        int bc = s.cand_c[tid][0];
        for (int k = 1; k < 16; ++k) {
            const double dd = s.cand_d[tid][k];
            const int cc = s.cand_c[tid][k];
            if (dd < bd || (dd == bd && cc < bc)) { bd = dd; bc = cc; }
        }
        store(row(tid), bc);
    }
}

__global__ __launch_bounds__(256) void assign_f64_kernel(const float *__restrict__ coarse, int K, int d,
                                                         const float *__restrict__ x, int64_t ldx, int64_t n,
                                                         int32_t *__restrict__ cells, int scale, int accumulate)
{
    __shared__ AssignTile s;
    const int64_t i0 = (int64_t)blockIdx.x * ASG_TM;
    assign_tile(s, coarse, K, d, x + i0 * ldx, ldx, [&](int k) { return i0 + k < n ? k : -1; },
                [&](int k, int bc) { cells[i0 + k] = (accumulate ? cells[i0 + k] : 0) + bc * scale; });
}

// ------------------------------------------------------------------ what the filter leaves

// A vector that the filter cannot decide is marked in `cells`: what the pass found there (0 without `accumulate`) with
// bit 30 turned over.  No cell looks like that: cells are below 2^28 where they accumulate and below 2^30 otherwise (the
// filter takes no more centroids), or, for a vector with a NaN, 0x7fffffff times the scale plus a cell.
constexpr int ASG_MARK = 0x40000000;
constexpr int ASG_MARK_MAX_K = 1 << 30;

__device__ __forceinline__ bool assign_marked(int cell, int K, int accumulate)
{
    const int was = cell ^ ASG_MARK;
    return accumulate ? (unsigned)was < (1u << 28) || was == (int)(0x7fffffffu * (unsigned)K) : was == 0;
}

// Every workgroup looks for the marks of `range` vectors (a multiple of ASG_TM, up to ASG_RANGE) and measures those
// vectors against all cells, by the definition: 128 at a time in tiles, or, of a few, four at a time and a lane per
// cell (a tile takes as long as five such rounds whatever it holds).  The filter's own last steps were slower at it, and
// cost the filter its registers.  Ranges rather than single tiles, so that few marks fill few tiles; 512 workgroups.
constexpr int ASG_RANGE = 4096, ASG_FEW = 20;

__global__ __launch_bounds__(256) void assign_rest_kernel(const float *__restrict__ coarse, int K, int d,
                                                          const float *__restrict__ x, int64_t ldx, int64_t n, int range,
                                                          int32_t *__restrict__ cells, int scale, int accumulate)
{
    __shared__ AssignTile s;
    __shared__ uint16_t todo[ASG_RANGE];
    __shared__ int ntodo;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t i0 = (int64_t)blockIdx.x * range;
    if (tid == 0) ntodo = 0;
    __syncthreads();
    for (int k = tid; k < range; k += 256) {
        const bool found = i0 + k < n && assign_marked(cells[i0 + k], K, accumulate);
        if (found) todo[atomicAdd(&ntodo, 1)] = (uint16_t)k;
    }
    __syncthreads();
    const int count = ntodo;
    auto store = [&](int k, int bc) { cells[i0 + k] = (cells[i0 + k] ^ ASG_MARK) + bc * scale; };
    const int few = d <= 4 ? ASG_RANGE : ASG_FEW;  // (a tile computes 16 components at least)
    int k0 = 0;
    for (; count - k0 > few; k0 += ASG_TM) {  // uniform
        assign_tile(s, coarse, K, d, x + i0 * ldx, ldx, [&](int k) { return k0 + k < count ? (int)todo[k0 + k] : -1; }, store);
        __syncthreads();
    }
    double(&red_d)[16][4] = *reinterpret_cast<double(*)[16][4]>(s.cand_d);
    int(&red_c)[16][4] = *reinterpret_cast<int(*)[16][4]>(s.cand_c);
    for (; k0 < count; k0 += 4) {  // uniform
        const float *xr[4];
        double bd[4];
        int bc[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            xr[k] = x + (i0 + todo[min(k0 + k, count - 1)]) * ldx;
            bd[k] = __builtin_inf();
            bc[k] = 0x7fffffff;
        }
        for (int c = tid; c < K; c += 256) {
            const float *cr = coarse + (size_t)c * d;
            double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
            for (int t = 0; t < d; ++t) {
                const double cv = (double)cr[t];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const double df = (double)xr[k][t] - cv;
                    acc[k] = fma(df, df, acc[k]);
                }
            }
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (acc[k] < bd[k] || (acc[k] == bd[k] && c < bc[k])) { bd[k] = acc[k]; bc[k] = c; }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
#pragma unroll
            for (int m = 32; m >= 1; m >>= 1) {
                const double od = __shfl_xor(bd[k], m);
                const int oc = __shfl_xor(bc[k], m);
                if (od < bd[k] || (od == bd[k] && oc < bc[k])) { bd[k] = od; bc[k] = oc; }
            }
            if (lane == 0) { red_d[wave][k] = bd[k]; red_c[wave][k] = bc[k]; }
        }
        __syncthreads();
        if (tid < 4 && k0 + tid < count) {
            double d0 = red_d[0][tid];
            int c0 = red_c[0][tid];
            for (int w = 1; w < 4; ++w)
                if (red_d[w][tid] < d0 || (red_d[w][tid] == d0 && red_c[w][tid] < c0)) {
                    d0 = red_d[w][tid];
                    c0 = red_c[w][tid];
                }
            store(todo[k0 + tid], c0);
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------------ filter on the matrix units

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int AF_MAX_D = 256;

// hi + lo = v to 2^-18 relative
__device__ __forceinline__ void split_bf16(const f32x8 v, bf16x8 *hi, bf16x8 *lo)
{
    *hi = __builtin_convertvector(v, bf16x8);
    *lo = __builtin_convertvector(v - __builtin_convertvector(*hi, f32x8), bf16x8);
}

// eight consecutive components t .. t+7 of a row, zero at and beyond d
template <bool VEC>
__device__ __forceinline__ f32x8 load8(const float *row, int t, int d)
{
    f32x8 v;
    if constexpr (VEC) {  // 16-byte aligned rows of whole steps
        const float4 a = *reinterpret_cast<const float4 *>(row + t);
        const float4 b = *reinterpret_cast<const float4 *>(row + t + 4);
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
        v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = t + e < d ? row[t + e] : 0.0f;
    }
    return v;
}

// NT: threads.  KS: steps of 16 components (16 KS >= d).  NB: blocks of 32 vectors per wavefront.  VEC: 16 KS = d, and
// the rows of x and of the centroids start on 16-byte boundaries.
template <int NT, int KS, int NB, bool VEC>
__global__ __launch_bounds__(NT, 2) void assign_filter_kernel(const float *__restrict__ coarse, int K, int d,
                                                                 const float *__restrict__ x, int64_t ldx,
                                                                 int64_t n, int32_t *__restrict__ cells, int scale,
                                                                 int accumulate)
{
    constexpr int PS = KS <= 4 ? 4 : 8;     // threads that split one centroid at a time
    constexpr int IT = (KS + PS - 1) / PS;  // steps of 16 components per thread
    constexpr int NW = NT / WAVE;
    constexpr int TC = NT / PS;             // cells per tile
    constexpr int CT = TC / 32;
    constexpr int TM = NW * NB * 32;        // vectors per workgroup
    static_assert(TC % 32 == 0 && KS <= PS * IT, "");
    // A tile of centroids as the matrix instructions read them: step s, part (hi, lo), lane, 16 bytes
    __shared__ __attribute__((aligned(16))) bf16x8 tile[2][CT][KS][2][WAVE];
    __shared__ __attribute__((aligned(16))) float nrm[2][TC];
    __shared__ __attribute__((aligned(16))) float ref[16 * KS];
    __shared__ float cmax_s[NW];
    __shared__ int cand[TM][4];     // groups to measure, -1: none
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 31, half = lane >> 5;
    const int64_t i0 = (int64_t)blockIdx.x * TM;

    // The reference: per component, the middle of eight centroids of the range.  (Any vector would do; one amid the
    // centroids keeps the norms, and with them the margins, small, and a few stray or non-finite ones do not move this.)
    for (int t = tid; t < 16 * KS; t += NT) {
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
        ref[t] = 0.5f * v[3] + 0.5f * v[4];
    }
    __syncthreads();

    // this wavefront's vectors: operand -2 x', split; lane (col, half) holds components 16 s + 8 half ..
    bf16x8 bh[NB][KS], bl[NB][KS];
    float xn[NB];  // |x'|^2
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int64_t i = i0 + (wave * NB + nb) * 32 + col;
        const float *row = x + (i < n ? i : 0) * ldx;
        float s2 = 0.0f;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int t = 16 * s + 8 * half;
            f32x8 v = load8<VEC>(row, t, d);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                v[e] = v[e] - ref[t + e];  // (zero beyond d)
                s2 = __builtin_fmaf(v[e], v[e], s2);
                v[e] = v[e] * -2.0f;
            }
            split_bf16(v, &bh[nb][s], &bl[nb][s]);
        }
        xn[nb] = s2 + __shfl_xor(s2, 32);
    }

    // Rounding of a score, whatever the unit: |score - (distance^2 - |x'|^2)| <= eps (|x'|^2 + |c'|^2), with D = 16 KS:
    // the differences 4 2^-24; what the splits and the missing lo.lo leave out 3.1 2^-18; 3 D + 1 additions of values
    // up to 2 (|x'|^2 + |c'|^2) (3 D + 1) 2^-22 (2^-23 each: no assumption on how the matrix units round); the norms
    // (D + 8) 2^-24; 1.28e-5 + 7.8e-7 D in all.  The part of the centroid comes off its score from the start, so that a
    // far centroid loosens its own score and no other's.
    constexpr float eps = 1.5e-5f + 9e-7f * (16 * KS);

    // thread -> centroid and steps it splits: eight neighbouring lanes hold eight centroids (their
    // 16-byte LDS writes are contiguous), a centroid's threads lie in one wavefront
    const int crow = (tid & 7) + 8 * (tid / (8 * PS));
    const int part = (tid >> 3) % PS;
    f32x8 raw[IT][2];
    auto fetch = [&](int c0) {
        const float *row = coarse + (size_t)min(c0 + crow, K - 1) * d;
#pragma unroll
        for (int it = 0; it < IT; ++it)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                if (part + PS * it < KS) raw[it][h] = load8<VEC>(row, 16 * (part + PS * it) + 8 * h, d);
    };
    float cmax = 0.0f;
    auto stash = [&](int c0, int buf) {
        float s2 = 0.0f;
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int s = part + PS * it;
            if (s < KS) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const float4 r0 = *reinterpret_cast<const float4 *>(&ref[16 * s + 8 * h]);
                    const float4 r1 = *reinterpret_cast<const float4 *>(&ref[16 * s + 8 * h + 4]);
                    f32x8 v = raw[it][h];
                    v[0] -= r0.x; v[1] -= r0.y; v[2] -= r0.z; v[3] -= r0.w;
                    v[4] -= r1.x; v[5] -= r1.y; v[6] -= r1.z; v[7] -= r1.w;
#pragma unroll
                    for (int e = 0; e < 8; ++e) s2 = __builtin_fmaf(v[e], v[e], s2);
                    bf16x8 hi, lo;
                    split_bf16(v, &hi, &lo);
                    tile[buf][crow >> 5][s][0][h * 32 + (crow & 31)] = hi;
                    tile[buf][crow >> 5][s][1][h * 32 + (crow & 31)] = lo;
                }
            }
        }
#pragma unroll
        for (int m = 8; m < 8 * PS; m <<= 1) s2 += __shfl_xor(s2, m);
        const bool in = c0 + crow < K;
        if (in) cmax = fmaxf(cmax, s2);  // (NaN: left out)
        if (part == 0) nrm[buf][crow] = in ? s2 * (1.0f - eps) : __builtin_inff();
    };

    float b1[NB], b2[NB], b3[NB];  // the three smallest group minima, ascending; the groups of the first two
    int a1[NB], a2[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        b1[nb] = b2[nb] = b3[nb] = __builtin_inff();
        a1[nb] = a2[nb] = 0;
    }
    fetch(0);
    stash(0, 0);
    __syncthreads();
    int buf = 0;
    for (int c0 = 0; c0 < K; c0 += TC, buf ^= 1) {
        if (c0 + TC < K) fetch(c0 + TC);  // uniform; travels while this tile is multiplied
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            // result (cell 8 (r / 4) + 4 half + r % 4, vector col) starts at |c'|^2
            f32x16 init;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float4 v = *reinterpret_cast<const float4 *>(&nrm[buf][ct * 32 + 8 * g + 4 * half]);
                init[4 * g] = v.x; init[4 * g + 1] = v.y; init[4 * g + 2] = v.z; init[4 * g + 3] = v.w;
            }
            f32x16 acc[NB];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) acc[nb] = init;
            // (the operands of a step are requested two steps ahead)
            bf16x8 a[3][2];
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                a[s][0] = tile[buf][ct][s][0][lane];
                a[s][1] = tile[buf][ct][s][1][lane];
            }
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                if (s + 2 < KS) {
                    a[(s + 2) % 3][0] = tile[buf][ct][s + 2][0][lane];
                    a[(s + 2) % 3][1] = tile[buf][ct][s + 2][1][lane];
                }
                const bf16x8 ah = a[s % 3][0], al = a[s % 3][1];
                __builtin_amdgcn_sched_barrier(0);  // (left to itself the compiler requests them where they are used)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bh[nb][s], acc[nb], 0, 0, 0);
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bh[nb][s], acc[nb], 0, 0, 0);
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bl[nb][s], acc[nb], 0, 0, 0);
            }
            const int g = c0 / 32 + ct;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                float v = fminf(acc[nb][0], acc[nb][1]);
#pragma unroll
                for (int r = 2; r < 16; ++r) v = fminf(v, acc[nb][r]);
                const bool l1 = v < b1[nb], l2 = v < b2[nb];
                b3[nb] = fminf(b3[nb], fmaxf(b2[nb], v));
                b2[nb] = fminf(b2[nb], fmaxf(b1[nb], v));
                b1[nb] = fminf(b1[nb], v);
                const int second = l2 ? g : a2[nb];
                a2[nb] = l1 ? a1[nb] : second;
                a1[nb] = l1 ? g : a1[nb];
            }
        }
        if (c0 + TC < K) stash(c0 + TC, buf ^ 1);  // uniform; that buffer was read before the last barrier
        __syncthreads();
    }

    // largest |c'|^2
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) cmax = fmaxf(cmax, __shfl_xor(cmax, m));
    if (lane == 0) cmax_s[wave] = cmax;
    __syncthreads();
    cmax = cmax_s[0];
    for (int k = 1; k < NW; ++k) cmax = fmaxf(cmax, cmax_s[k]);

    // With b1 the smallest score, reached by a cell c*: the closest cell's score is at most b1 + 2 eps (|x'|^2 + |c*'|^2).
    // |c*'|^2 is at most the largest of all cells, and |c*'| <= |x'| + |x' - c*'| with |x' - c*'|^2 <= b1 + |x'|^2 + what
    // rounding adds, under a thousandth of |x'|^2.  A centroid whose score overflows or is NaN (it loses every
    // comparison) is not the closest to a vector that has one within 1e18.
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int v = (wave * NB + nb) * 32 + col;
        const float low = fminf(b1[nb], __shfl_xor(b1[nb], 32));
        const float far = __builtin_sqrtf(xn[nb]) + __builtin_sqrtf(fmaxf(low + xn[nb], 0.0f) + 1e-3f * xn[nb]);
        const float thr = low + __builtin_fmaf(2.0f * eps, xn[nb] + 1.01f * fminf(far * far, cmax), 1e-30f);
        // (comparisons that a NaN fails)
        const bool sure = xn[nb] < 1e36f && thr < 1e36f && b3[nb] > thr;
        // this lane's groups in question, then those of the other half; the first entry is never empty
        // unless the vector is left to the kernel after this one
        const int g1 = b1[nb] <= thr ? 2 * a1[nb] + half : -1, g2 = b2[nb] <= thr ? 2 * a2[nb] + half : -1;
        const int o1 = __shfl_xor(g1, 32), o2 = __shfl_xor(g2, 32);
        const int other = __shfl_xor((int)sure, 32);  // (asked by all lanes: a lane that does not ask gives nothing)
        const bool all = !(sure && other);
        if (half == 0) {
            cand[v][0] = all ? -2 : g1 >= 0 ? g1 : o1;
            cand[v][1] = g1 >= 0 ? g2 : o2;
            cand[v][2] = g1 >= 0 ? o1 : -1;
            cand[v][3] = g1 >= 0 ? o2 : -1;
            if (all && i0 + v < n) cells[i0 + v] = (accumulate ? cells[i0 + v] : 0) ^ ASG_MARK;
        }
    }
    __syncthreads();

    // The groups in question, 16 lanes per vector: the 16 distances of a group in float32, the lanes side by side along
    // the components (a lane per cell would read 64 different lines per load).  A cell that no other comes within the
    // rounding of is the closest; else the cells that do are measured by the definition, a lane each.
    const int r = tid & 15, team = (lane >> 4) * 16;
    auto cell_of = [&](int g, int k) { return (g >> 1) * 32 + 8 * (k >> 2) + 4 * (g & 1) + (k & 3); };
    for (int v = tid >> 4; v < TM; v += NT / 16) {
        const int64_t i = i0 + v;
        if (i >= n || cand[v][0] < 0) continue;  // uniform over the 16 lanes
        const float *xr = x + i * ldx;
        float xv[KS];
        constexpr int W = VEC && KS % 4 == 0 ? 4 : 1;  // components per load
#pragma unroll
        for (int e = 0; e < KS / W; ++e)
#pragma unroll
            for (int u = 0; u < W; ++u) {
                const int t = W * (r + 16 * e) + u;
                xv[W * e + u] = VEC || t < d ? xr[t] : 0.0f;
            }
        // distance to cell r of group g
        auto measure = [&](int g) {
            float part[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const float *cr = coarse + (size_t)min(cell_of(g, k), K - 1) * d;
                float acc = 0.0f;
#pragma unroll
                for (int e = 0; e < KS / W; ++e) {
                    float cv[W];
                    if constexpr (W == 4) {
                        const float4 f = *reinterpret_cast<const float4 *>(cr + 4 * (r + 16 * e));
                        cv[0] = f.x; cv[1] = f.y; cv[2] = f.z; cv[3] = f.w;
                    } else {
                        const int t = r + 16 * e;
                        cv[0] = VEC || t < d ? cr[t] : 0.0f;
                    }
#pragma unroll
                    for (int u = 0; u < W; ++u) {
                        const float df = xv[W * e + u] - cv[u];
                        acc = __builtin_fmaf(df, df, acc);
                    }
                }
                part[k] = acc;
            }
            // sums over the 16 lanes, halving the cells a lane is responsible for: lane r ends with cell r
#pragma unroll
            for (int w = 8; w >= 1; w >>= 1)
#pragma unroll
                for (int k = 0; k < w; ++k) {
                    const bool up = r & w;
                    const float keep = up ? part[k + w] : part[k], give = up ? part[k] : part[k + w];
                    part[k] = keep + __shfl_xor(give, w);
                }
            return cell_of(g, r) < K && part[0] == part[0] ? part[0] : __builtin_inff();  // (a NaN is never the closest)
        };
        auto lowest = [&](float f) {
#pragma unroll
            for (int w = 8; w >= 1; w >>= 1) f = fminf(f, __shfl_xor(f, w));
            return f;
        };
        // rounding of two sums of d squares (d / 16 + 4 additions, the differences, the squares): (d / 8 + 14) 2^-24,
        // here at least 1.3 times that
        auto slack = [&](float f) { return f + __builtin_fmaf(f, 2e-6f + 1e-7f * KS, 1e-33f); };
        auto among = [&](bool near) { return __popcll((__ballot(near) >> team) & 0xffffull); };
        const int g0 = cand[v][0];
        const bool more = cand[v][1] >= 0 || cand[v][2] >= 0 || cand[v][3] >= 0;  // uniform over the 16 lanes
        float dist[4] = {measure(g0), __builtin_inff(), __builtin_inff(), __builtin_inff()};
        float close = slack(lowest(dist[0]));
        int rivals = among(dist[0] <= close);
        int bc = dist[0] <= close ? cell_of(g0, r) : 0x7fffffff;
        if (more) {
#pragma unroll 1
            for (int q = 1; q < 4; ++q) {
                const int g = cand[v][q];
                if (g < 0) continue;  // uniform over the 16 lanes
                const float to = measure(g);
#pragma unroll
                for (int p = 1; p < 4; ++p) dist[p] = p == q ? to : dist[p];
            }
            close = slack(lowest(fminf(fminf(dist[0], dist[1]), fminf(dist[2], dist[3]))));
            bc = 0x7fffffff;
            rivals = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const bool near = dist[q] <= close && cand[v][q] >= 0;
                rivals += among(near);
                if (near) bc = cell_of(cand[v][q], r);
            }
        }
        if (rivals > 1) {  // uniform over the 16 lanes
            double bd = __builtin_inf();
            bc = 0x7fffffff;
#pragma unroll 1
            for (int q = 0; q < 4; ++q) {
                const int g = cand[v][q];
                const float dq = q == 0 ? dist[0] : q == 1 ? dist[1] : q == 2 ? dist[2] : dist[3];
                const int c = cell_of(g, r);
                if (g < 0 || !(dq <= close) || c >= K) continue;
                const float *cr = coarse + (size_t)c * d;
                double dd = 0.0;
                auto add = [&](float a, float b) {
                    const double df = (double)a - (double)b;
                    dd = fma(df, df, dd);
                };
                if constexpr (VEC) {
#pragma unroll 4
                    for (int t = 0; t < d; t += 4) {
                        const float4 a = *reinterpret_cast<const float4 *>(xr + t), b = *reinterpret_cast<const float4 *>(cr + t);
                        add(a.x, b.x); add(a.y, b.y); add(a.z, b.z); add(a.w, b.w);
                    }
                } else {
#pragma unroll 8
                    for (int t = 0; t < d; ++t) add(xr[t], cr[t]);
                }
                if (dd < bd || (dd == bd && c < bc)) { bd = dd; bc = c; }
            }
#pragma unroll
            for (int w = 8; w >= 1; w >>= 1) {
                const double od = __shfl_xor(bd, w);
                const int oc = __shfl_xor(bc, w);
                if (od < bd || (od == bd && oc < bc)) { bd = od; bc = oc; }
            }
        } else {
#pragma unroll
            for (int w = 8; w >= 1; w >>= 1) bc = min(bc, __shfl_xor(bc, w));
        }
        if (r == 0) cells[i] = (accumulate ? cells[i] : 0) + bc * scale;
    }
}

// ------------------------------------------------------------------ host

template <int KS>
static void launch_filter(const float *coarse, int K, int d, const float *x, int64_t ldx, int64_t n, int32_t *cells,
                          int scale, int accumulate, hipStream_t st)
{
    const bool vec = d == 16 * KS && ldx % 4 == 0 && ((uintptr_t)coarse & 15) == 0 && ((uintptr_t)x & 15) == 0;
    if constexpr (KS <= 8)
        if (vec && n >= 512 * 256) {  // 512 vectors per workgroup once that fills the chip; else 128
            hipLaunchKernelGGL((assign_filter_kernel<512, KS, 2, true>), dim3((unsigned)ceil_div(n, 512)), dim3(512), 0,
                               st, coarse, K, d, x, ldx, n, cells, scale, accumulate);
            return;
        }
    const dim3 grid((unsigned)ceil_div(n, 128));
    if (vec)
        hipLaunchKernelGGL((assign_filter_kernel<256, KS, 1, true>), grid, dim3(256), 0, st, coarse, K, d, x, ldx, n,
                           cells, scale, accumulate);
    else
        hipLaunchKernelGGL((assign_filter_kernel<256, KS, 1, false>), grid, dim3(256), 0, st, coarse, K, d, x, ldx, n,
                           cells, scale, accumulate);
}

// cells[i] = (accumulate ? cells[i] : 0) + scale * (closest of K centroids to the d components at x + i ldx)
static int assign_pass(const float *coarse, int K, int d, const float *x, int64_t ldx, int64_t n, int32_t *cells,
                       int scale, int accumulate, hipStream_t st)
{
    const bool filter = d <= AF_MAX_D && K <= ASG_MARK_MAX_K;
    if (!filter)
        hipLaunchKernelGGL(assign_f64_kernel, dim3((unsigned)ceil_div(n, ASG_TM)), dim3(256), 0, st, coarse, K, d, x,
                           ldx, n, cells, scale, accumulate);
    else if (d <= 32)
        launch_filter<2>(coarse, K, d, x, ldx, n, cells, scale, accumulate, st);
    else if (d <= 64)
        launch_filter<4>(coarse, K, d, x, ldx, n, cells, scale, accumulate, st);
    else if (d <= 96)
        launch_filter<6>(coarse, K, d, x, ldx, n, cells, scale, accumulate, st);
    else if (d <= 128)
        launch_filter<8>(coarse, K, d, x, ldx, n, cells, scale, accumulate, st);
    else
        launch_filter<16>(coarse, K, d, x, ldx, n, cells, scale, accumulate, st);
    if (filter) {
        const int64_t range = std::min<int64_t>(ASG_RANGE, std::max<int64_t>(512, ceil_div(ceil_div(n, 512), ASG_TM) * ASG_TM));
        hipLaunchKernelGGL(assign_rest_kernel, dim3((unsigned)ceil_div(n, range)), dim3(256), 0, st, coarse, K, d, x, ldx, n,
                           (int)range, cells, scale, accumulate);
    }
    QADC_HIP_TRY(hipGetLastError());
    return QADC_OK;
}

int ivf_assign(const float *coarse, int K, int d, const float *x, int64_t n, int32_t *cells, hipStream_t st)
{
    if (K < 1 || d < 1 || n < 0)
        return fail(QADC_EINVAL, "qadc_ivf_assign: K=%d d=%d n=%lld", K, d, (long long)n);
    if (n == 0) return QADC_OK;
    if (!coarse || !x || !cells) return fail(QADC_EINVAL, "qadc_ivf_assign: null pointer");
    if (ceil_div(n, ASG_TM) > 0x7fffffffll) return fail(QADC_EINVAL, "qadc_ivf_assign: n too large for one call");
    return assign_pass(coarse, K, d, x, d, n, cells, 1, 0, st);
}

// Cells of an inverted multi-index: the coarse quantizer is the product of two quantizers of K
// centroids over the two halves of the vector, cell = K * (closest of halves[0] to the first half)
// + (closest of halves[1] to the second half).  Two passes of the assignment over the halves of the
// rows of x.
int multi_index_assign(const float *halves, int K, int d, const float *x, int64_t n, int32_t *cells,
                       hipStream_t st)
{
    if (K < 1 || K > 16384 || d < 2 || (d & 1) || n < 0)
        return fail(QADC_EINVAL, "qadc_multi_index_assign: K=%d d=%d n=%lld", K, d, (long long)n);
    if (n == 0) return QADC_OK;
    if (!halves || !x || !cells) return fail(QADC_EINVAL, "qadc_multi_index_assign: null pointer");
    if (ceil_div(n, ASG_TM) > 0x7fffffffll)
        return fail(QADC_EINVAL, "qadc_multi_index_assign: n too large for one call");
    const int dh = d / 2;
    const int rc = assign_pass(halves, K, dh, x, d, n, cells, K, 0, st);
    if (rc != QADC_OK) return rc;
    return assign_pass(halves + (size_t)K * dh, K, dh, x + dh, d, n, cells, 1, 1, st);
}

}  // namespace qadc
