// Cell of a vector on gfx950 (Section 2.2 of the paper): cell(x) = index of the closest coarse centroid,
// float64 distances from the differences (one fused multiply-add per component, increasing component),
// the lowest cell among equal distances -- the vector quantizer q_i of the inverted index.
//
// assign_filter_kernel (d <= 256) finds that cell without forming all n x K float64 distances.  With x' and
// c' the differences to a reference vector, |x - c|^2 = |x'|^2 + |c'|^2 - 2 x'.c', and the part that depends
// on the cell is a matrix product: both factors are split into two bfloat16 numbers (16 significant bits)
// and hi.hi + hi.lo + lo.hi is summed in float32 by the matrix units.  A lane keeps, per vector, the three
// smallest of its group minima (a group: the 16 cells of a result tile that lie in one lane).  Whatever the
// rounding, the closest cell lies in a group whose minimum is within `margin` (bound below) of the smallest;
// those groups -- mostly one -- are measured in float64 by the definition, and a vector that may have more of
// them than a lane remembers (equal centroids, values beyond the float32 range, infinities, NaN) is measured
// against all cells.  The result is the definition's, whatever the route.
//
// Bound: 3 x 2 n K d operations on the matrix units.  Measured for 1 M vectors, d = 128, K = 4096: 2.9 ms =
// 1.1 PFLOP/s of bfloat16 products (the float64 kernel: 37.8 ms); 2.0 ms of it are products and group minima,
// 0.4 splitting the centroids, which every workgroup does again -- so eight wavefronts share the tiles and keep
// the operands of 64 vectors each in registers for the whole walk -- and 0.5 the last step.
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

// Thread (tx, ty), tx = tid & 15, ty = tid >> 4, owns the vectors 8*ty .. 8*ty+7 of the tile and
// the cells 32*k + 2*tx + e (k < 4, e < 2): a wavefront's 16-byte reads of the cells are
// contiguous across its lanes, its reads of the vectors are the same for 16 lanes.
__global__ __launch_bounds__(256) void assign_f64_kernel(const float *__restrict__ coarse, int K, int d,
                                                         const float *__restrict__ x, int64_t ldx, int64_t n,
                                                         int32_t *__restrict__ cells, int scale, int accumulate)
{
    __shared__ __attribute__((aligned(16))) double xs[ASG_TK][ASG_LD];
    __shared__ __attribute__((aligned(16))) double cs[ASG_TK][ASG_LD];
    __shared__ double cand_d[ASG_TM][16];
    __shared__ int cand_c[ASG_TM][16];
    const int tid = threadIdx.x;
    const int tx = tid & 15, ty = tid >> 4;
    const int64_t i0 = (int64_t)blockIdx.x * ASG_TM;
    double best_d[8];
    int best_c[8];
#pragma unroll
    for (int a = 0; a < 8; ++a) { best_d[a] = __builtin_inf(); best_c[a] = 0x7fffffff; }

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
                const int row = idx >> 4, col = idx & 15;
                const int t = t0 + col;
                const int64_t i = i0 + row;
                const int c = c0 + row;
                xs[col][row] = (i < n && t < d) ? (double)x[i * ldx + t] : 0.0;
                cs[col][row] = (c < K && t < d) ? (double)coarse[(size_t)c * d + t] : 0.0;
            }
            __syncthreads();
#pragma unroll 4
            for (int kk = 0; kk < ASG_TK; ++kk) {
                double xv[8], cv[8];
#pragma unroll
                for (int a = 0; a < 8; a += 2) {
                    const double2 v = *reinterpret_cast<const double2 *>(&xs[kk][8 * ty + a]);
                    xv[a] = v.x; xv[a + 1] = v.y;
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const double2 v = *reinterpret_cast<const double2 *>(&cs[kk][32 * k + 2 * tx]);
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
        cand_d[8 * ty + a][tx] = best_d[a];
        cand_c[8 * ty + a][tx] = best_c[a];
    }
    __syncthreads();
    if (tid < ASG_TM) {
        const int64_t i = i0 + tid;
        if (i < n) {
            double bd = cand_d[tid][0];
            int bc = cand_c[tid][0];
            for (int k = 1; k < 16; ++k) {
                const double dd = cand_d[tid][k];
                const int cc = cand_c[tid][k];
                if (dd < bd || (dd == bd && cc < bc)) { bd = dd; bc = cc; }
            }
            cells[i] = (accumulate ? cells[i] : 0) + bc * scale;
        }
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
    __shared__ int redo[TM];        // vectors to measure against all cells
    __shared__ int nredo;
    __shared__ double red_d[4][NW];  // [vector of four][wavefront]
    __shared__ int red_c[4][NW];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 31, half = lane >> 5;
    const int64_t i0 = (int64_t)blockIdx.x * TM;

    // the reference: the mean of eight centroids of the range (any vector would do; one amid the
    // centroids keeps the norms, and with them the margin, small)
    for (int t = tid; t < 16 * KS; t += NT) {
        float s = 0.0f;
        if (t < d)
            for (int k = 0; k < 8; ++k) s += coarse[(size_t)((int64_t)k * K >> 3) * d + t];
        ref[t] = s * 0.125f;
    }
    if (tid == 0) nredo = 0;
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
        if (in) cmax = s2 > cmax || s2 != s2 ? s2 : cmax;  // (a NaN stays: it makes every margin NaN)
        if (part == 0) nrm[buf][crow] = in ? s2 : __builtin_inff();
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
    for (int m = 32; m >= 1; m >>= 1) {
        const float o = __shfl_xor(cmax, m);
        cmax = o > cmax || o != o ? o : cmax;
    }
    if (lane == 0) cmax_s[wave] = cmax;
    __syncthreads();
    cmax = cmax_s[0];
    for (int k = 1; k < NW; ++k) cmax = cmax_s[k] > cmax || cmax_s[k] != cmax_s[k] ? cmax_s[k] : cmax;

    // Bound of |score - (exact distance - |x'|^2)|, with S = |x'|^2 + max |c'|^2 >= 2 |x'| |c'| and D = 16 KS:
    // rounding of the differences 4 S 2^-24; what the splits and the missing lo.lo leave out 3.1 S 2^-18; 3 D + 1
    // additions of the product 2 S (3 D + 1) 2^-23 (2^-23: no assumption on how the matrix units round); the
    // norms S (D + 8) 2^-24.  The margin is twice that for two candidates, rounded up.
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int v = (wave * NB + nb) * 32 + col;
        const float S = xn[nb] + cmax;
        const float margin = __builtin_fmaf(S, 3e-5f + 1.8e-6f * (16 * KS), 1e-30f);
        const float thr = fminf(b1[nb], __shfl_xor(b1[nb], 32)) + margin;
        // (comparisons that a NaN fails)
        const bool sure = S < 1e37f && thr < 1e37f && b3[nb] > thr;
        // this lane's groups in question, then those of the other half; the first entry is never empty
        // unless the vector has to be measured against all cells
        const int g1 = b1[nb] <= thr ? 2 * a1[nb] + half : -1, g2 = b2[nb] <= thr ? 2 * a2[nb] + half : -1;
        const int o1 = __shfl_xor(g1, 32), o2 = __shfl_xor(g2, 32);
        const int other = __shfl_xor((int)sure, 32);  // (asked by all lanes: a lane that does not ask gives nothing)
        const bool all = !(sure && other);
        if (half == 0) {
            cand[v][0] = all ? -2 : g1 >= 0 ? g1 : o1;
            cand[v][1] = g1 >= 0 ? g2 : o2;
            cand[v][2] = g1 >= 0 ? o1 : -1;
            cand[v][3] = g1 >= 0 ? o2 : -1;
            if (all && i0 + v < n) redo[atomicAdd(&nredo, 1)] = v;
        }
    }
    __syncthreads();

    // The groups in question, 16 lanes per vector.  One group: its 16 distances in float32, the lanes side by
    // side along the components (a lane per cell would read 64 different lines per load), and unless a second
    // one lies within the rounding of the closest that is the cell.  Otherwise by the definition, a lane per cell.
    const int r = tid & 15;
    auto cell_of = [&](int g, int k) { return (g >> 1) * 32 + 8 * (k >> 2) + 4 * (g & 1) + (k & 3); };
    for (int v = tid >> 4; v < TM; v += NT / 16) {
        const int64_t i = i0 + v;
        const int g0 = cand[v][0];
        if (i >= n || g0 < 0) continue;  // uniform over the 16 lanes
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
        float part[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const float *cr = coarse + (size_t)min(cell_of(g0, k), K - 1) * d;
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
        int bc = cell_of(g0, r);
        const bool in = bc < K;
        const float d0 = in ? part[0] : __builtin_inff();
        float d1 = d0, d2 = __builtin_inff();  // the two smallest of the 16 lanes (NaN: ignored here, caught below)
        int at = r;
#pragma unroll
        for (int w = 8; w >= 1; w >>= 1) {
            const float o1 = __shfl_xor(d1, w), o2 = __shfl_xor(d2, w);
            const int oa = __shfl_xor(at, w);
            d2 = fminf(fmaxf(d1, o1), fminf(d2, o2));
            at = o1 < d1 ? oa : at;
            d1 = fminf(d1, o1);
        }
        // rounding of two sums of d squares (d / 16 + 4 additions, the differences, the squares), doubled
        const float close = __builtin_fmaf(d1, 2e-6f + 1e-7f * KS, 1e-33f);
        if (cand[v][1] < 0 && cand[v][2] < 0 && cand[v][3] < 0 && d1 < 1e37f && d2 > d1 + close) {
            bc = cell_of(g0, at);
        } else {
            double bd = __builtin_inf();
            bc = 0x7fffffff;
            for (int e = 0; e < 4; ++e) {
                const int g = cand[v][e];
                if (g < 0 || cell_of(g, r) >= K) continue;
                const float *cr = coarse + (size_t)cell_of(g, r) * d;
                double dd = 0.0;
                for (int t = 0; t < d; ++t) {
                    const double df = (double)xr[t] - (double)cr[t];
                    dd = fma(df, df, dd);
                }
                if (dd < bd || (dd == bd && cell_of(g, r) < bc)) { bd = dd; bc = cell_of(g, r); }
            }
#pragma unroll
            for (int w = 8; w >= 1; w >>= 1) {
                const double od = __shfl_xor(bd, w);
                const int oc = __shfl_xor(bc, w);
                if (od < bd || (od == bd && oc < bc)) { bd = od; bc = oc; }
            }
        }
        if (r == 0) cells[i] = (accumulate ? cells[i] : 0) + bc * scale;
    }

    // vectors to measure against all cells, four at a time
    const int todo = nredo;
    for (int k0 = 0; k0 < todo; k0 += 4) {  // uniform
        const float *xr[4];
        double bd[4];
        int bc[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            xr[k] = x + (i0 + redo[min(k0 + k, todo - 1)]) * ldx;
            bd[k] = __builtin_inf();
            bc[k] = 0x7fffffff;
        }
        for (int c = tid; c < K; c += NT) {
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
            if (lane == 0) { red_d[k][wave] = bd[k]; red_c[k][wave] = bc[k]; }
        }
        __syncthreads();
        if (tid < 4 && k0 + tid < todo) {
            double d0 = red_d[tid][0];
            int c0 = red_c[tid][0];
            for (int w = 1; w < NW; ++w)
                if (red_d[tid][w] < d0 || (red_d[tid][w] == d0 && red_c[tid][w] < c0)) {
                    d0 = red_d[tid][w];
                    c0 = red_c[tid][w];
                }
            const int64_t i = i0 + redo[k0 + tid];
            cells[i] = (accumulate ? cells[i] : 0) + c0 * scale;
        }
        __syncthreads();
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
    if (d <= 32)
        launch_filter<2>(coarse, K, d, x, ldx, n, cells, scale, accumulate, st);
    else if (d <= 64)
        launch_filter<4>(coarse, K, d, x, ldx, n, cells, scale, accumulate, st);
    else if (d <= 96)
        launch_filter<6>(coarse, K, d, x, ldx, n, cells, scale, accumulate, st);
    else if (d <= 128)
        launch_filter<8>(coarse, K, d, x, ldx, n, cells, scale, accumulate, st);
    else if (d <= AF_MAX_D)
        launch_filter<16>(coarse, K, d, x, ldx, n, cells, scale, accumulate, st);
    else
        hipLaunchKernelGGL(assign_f64_kernel, dim3((unsigned)ceil_div(n, ASG_TM)), dim3(256), 0, st, coarse, K, d, x,
                           ldx, n, cells, scale, accumulate);
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
