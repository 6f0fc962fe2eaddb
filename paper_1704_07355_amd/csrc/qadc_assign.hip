// Cell of a vector on gfx950 (Section 2.2 of the paper): cell(x) = index of the closest coarse centroid,
// float64 distances from the differences (one fused multiply-add per component, increasing component),
// the lowest cell among equal distances -- the vector quantizer q_i of the inverted index.
//
// assign_filter_kernel (d <= 256) finds that cell without forming all n x K float64 distances.  With x' and
// c' the differences to a reference vector, |x - c|^2 = |x'|^2 + |c'|^2 - 2 x'.c', and the part that depends
// on the cell is a matrix product, summed in float32 by the matrix units.  Both factors are one binary16 number each (11
// significant bits; scaled by a power of two to the middle of its range), or, where that does not pay (half_factors_pay),
// split into two bfloat16 numbers (16 bits, hi.hi + hi.lo + lo.hi).  A lane keeps, per vector, the four
// smallest of its group minima (a group: four consecutive cells, whose scores lie in one lane), with the number of the group
// in the lowest bits of its minimum.  Whatever the
// rounding, the closest cell lies in a group whose minimum is within a margin (bound below) of the smallest;
// those groups -- mostly one -- are measured in float32 and, cells that come within its rounding of each other, in
// float64 by the definition.  A vector that may have more of them than a lane remembers (many equal or very close
// centroids), or that is out of the factors' reach, is marked, and assign_rest_kernel takes it through the filter with
// split factors (if it has not been), then measures what is still undecided (more than three equal centroids in a lane,
// infinities, NaN) against all cells.  The result is the definition's, whatever the route.
//
// Bound: 2 n K d operations on the matrix units, the conversion of the centroids (every workgroup does it again, so eight
// wavefronts share the tiles and hold the operands of 64 vectors each in registers for the whole walk) and the group minima;
// per 64 cells a wavefront takes 32 products of 32 cycles and 190 vector instructions of four, which run beside the products
// (a wavefront alone: 4 instructions beside a product cost it nothing, 8 a fifth) where they stand among them: the
// minima are those of the 32 cells before, the conversion that of the next tile, and all is one block of code.  1.05 M vectors,
// d = 128: 0.25 ms + 0.22 ms per 1024 centroids = 1.2 PFLOP/s; the first part is the vectors, read twice, and the groups measured
// at the end: groups of 16 cells, 8 KiB of centroids per vector from L2, made it 0.48 ms (K = 4096: 1.42 ms -> 1.13; d = 64
// 0.80 -> 0.67; 500 k, d = 256 2.24 -> 1.49; 200 k, d = 96, K = 1000 0.147 -> 0.094; 37.5 ms in float64).  Vectors and centroids
// of one Gaussian, where a few in a hundred vectors have rivals within the margin: 1.75 -> 1.38.  The minima of the same 32 cells and
// the conversion behind the products: 0.25 ms per 1024 centroids.  Not faster: the order of instructions given by hand
// (1.23 ms for 1.13), workgroups of 256 threads, two per compute unit (1.58).
// A margin is a matter of the vector and of the closest cells: a far or NaN centroid costs the other cells
// nothing.  The slow case: 4096 different centroids that are all within the margin of every vector, 200 k of them, d = 128: 9.9 ms; every
// centroid eight times 2.3 (copies are left out: list_cells).
//
// assign_f64_kernel (d > 256: the vectors no longer fit the registers): a workgroup of 256 threads takes 128
// vectors and walks over all cells 128 at a time; 16 components of both go through LDS as float64 per step,
// every thread accumulates 8 x 8 distances and keeps, per vector, the best of the cells it has seen; the 16
// threads of a vector compare their candidates at the end under the order (distance, cell).  Vector-ALU
// bound: 2 float64 operations per (vector, cell, component), three fifths of the float64 vector peak.  (The loads of the next
// step in registers meanwhile: 15 to 25 % slower, they spill.)

#include "qadc_common.h"
#include "qadc_half.h"

namespace qadc {

// ------------------------------------------------------------------ float64

constexpr int ASG_TM = 128;  // vectors per workgroup
constexpr int ASG_TN = 128;  // cells per step
constexpr int ASG_TK = 16;   // components per step
constexpr int ASG_LD = ASG_TM + 2;  // row stride in doubles: keeps 16-byte alignment, shifts the banks

struct AssignTile {
    __attribute__((aligned(16))) double xs[ASG_TK][ASG_LD];
    __attribute__((aligned(16))) double cs[ASG_TK][ASG_LD];
    uint64_t cand_d[ASG_TM][16];
    int cand_c[ASG_TM][16];
};
constexpr uint64_t ASG_NONE = 0x7ff0000000000001ull;  // one above the bits of infinity

// The cells of up to ASG_TM vectors, by a workgroup of 256 threads; row(k): the row of x that is vector k of the tile, -1
// for none; cell(k), increasing with k: the k-th of K cells.
// Thread (tx, ty), tx = tid & 15, ty = tid >> 4, owns the vectors 8*ty .. 8*ty+7 of the tile and
// the cells 32*k + 2*tx + e (k < 4, e < 2): a wavefront's 16-byte reads of the cells are
// contiguous across its lanes, its reads of the vectors are the same for 16 lanes.
template <typename Row, typename Cell, typename Store>
__device__ __forceinline__ void assign_tile(AssignTile &s, const float *__restrict__ coarse, int K, int d,
                                            const float *__restrict__ x, int64_t ldx, Row row, Cell cell, Store store)
{
    const int tid = threadIdx.x;
    const int tx = tid & 15, ty = tid >> 4;
    // the smallest distance so far as its bits, which order like the numbers (none is negative): a NaN is above the start,
    // infinity below it
    uint64_t best_d[8];
    int best_c[8];
    const float *xr[8];  // the rows this thread fetches from, at its component (some row where there is no vector)
#pragma unroll
    for (int a = 0; a < 8; ++a) {
        best_d[a] = ASG_NONE;
        best_c[a] = 0x7fffffff;
        xr[a] = x + max(row(ty + 16 * a), 0) * ldx + tx;
    }

    for (int c0 = 0; c0 < K; c0 += ASG_TN) {
        int from[8];  // cells this thread fetches
#pragma unroll
        for (int e = 0; e < 8; ++e) from[e] = cell(min(c0 + ty + 16 * e, K - 1));
        double acc[8][8];
#pragma unroll
        for (int a = 0; a < 8; ++a)
#pragma unroll
            for (int b = 0; b < 8; ++b) acc[a][b] = 0.0;
        for (int t0 = 0; t0 < d; t0 += ASG_TK) {
            // 128 x 16 elements of x and of the centroids, eight of each per thread, zero beyond the last component
            float xl[8], cl[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) xl[e] = cl[e] = 0.0f;
            if (t0 + tx < d) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    xl[e] = xr[e][t0];
                    cl[e] = coarse[(size_t)from[e] * d + t0 + tx];
                }
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                s.xs[tx][ty + 16 * e] = (double)xl[e];
                s.cs[tx][ty + 16 * e] = (double)cl[e];
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
        // the smaller distance wins, the lower cell among equal distances: a thread meets its cells in increasing order
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const int c = c0 + 32 * (b >> 1) + 2 * tx + (b & 1);
            const uint64_t beyond = c < K ? 0 : ~0ull;
#pragma unroll
            for (int a = 0; a < 8; ++a) {
                const uint64_t dist = __builtin_bit_cast(uint64_t, acc[a][b]) | beyond;
                const bool closer = dist < best_d[a];
                best_d[a] = closer ? dist : best_d[a];
                best_c[a] = closer ? c : best_c[a];
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
        uint64_t bd = s.cand_d[tid][0];
        int bc = s.cand_c[tid][0];
        for (int k = 1; k < 16; ++k) {
            const uint64_t dd = s.cand_d[tid][k];
            const int cc = s.cand_c[tid][k];
            if (dd < bd || (dd == bd && cc < bc)) { bd = dd; bc = cc; }
        }
        store(row(tid), bc == 0x7fffffff ? bc : cell(bc));
    }
}

__global__ __launch_bounds__(256) void assign_f64_kernel(const float *__restrict__ coarse, int K, int d,
                                                         const float *__restrict__ x, int64_t ldx, int64_t n,
                                                         int32_t *__restrict__ cells, int scale, int accumulate)
{
    __shared__ AssignTile s;
    const int64_t i0 = (int64_t)blockIdx.x * ASG_TM;
    assign_tile(s, coarse, K, d, x + i0 * ldx, ldx, [&](int k) { return i0 + k < n ? k : -1; }, [](int k) { return k; },
                [&](int k, int bc) { cells[i0 + k] = (accumulate ? cells[i0 + k] : 0) + bc * scale; });
}

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

// ------------------------------------------------------------------ filter on the matrix units

constexpr int AF_MAX_D = 256;
constexpr float AF_NONE = 0x1p127f;  // no score (its low bits may be replaced: it stays a number)

// hi + lo = v to 2^-18 relative
__device__ __forceinline__ void split_bf16(const f32x8 v, bits16x8 *hi, bits16x8 *lo)
{
    const bf16x8 h = __builtin_convertvector(v, bf16x8);
    *hi = __builtin_bit_cast(bits16x8, h);
    *lo = __builtin_bit_cast(bits16x8, __builtin_convertvector(v - __builtin_convertvector(h, f32x8), bf16x8));
}

// How the factors of the products are held.
//   Half: one binary16 number (11 significant bits) of the difference to the reference, scaled by a power of two.
//   Split: two bfloat16 numbers (16 significant bits, the range of float32), three products per component.
enum class Factors { Half, Split };

// NT: threads.  KS: steps of 16 components (16 KS >= d).  NB: blocks of 32 vectors per wavefront.  VEC: 16 KS = d, and
// the rows of x and of the centroids start on 16-byte boundaries.
template <int NT, int KS, int NB, Factors F>
struct FilterShape {
    static constexpr int PS = KS <= 2 ? 2 : KS <= 4 ? 4 : 8;     // threads that convert one centroid at a time
    static constexpr int IT = (KS + PS - 1) / PS;  // steps of 16 components per thread
    static constexpr int NW = NT / WAVE;
    static constexpr int TC = NT / PS;             // cells per tile
    static constexpr int CT = TC / 32;
    static constexpr int TM = NW * NB * 32;        // vectors per workgroup
    static constexpr int PARTS = F == Factors::Split ? 2 : 1;
    // cells after which the groups found are given their numbers and merged with those before (a multiple of the tile)
    static constexpr int SEG = F == Factors::Split ? 512 : 4096;
    static constexpr unsigned MASK = SEG / 8 - 1;  // low bits of a group's minimum that hold its number in the segment
    static_assert(TC % 32 == 0 && SEG % TC == 0 && KS <= PS * IT, "");
};

template <int NT, int KS, int NB, Factors F>
struct FilterTile {
    using S = FilterShape<NT, KS, NB, F>;
    // A tile of centroids as the matrix instructions read them: step s, part (hi, lo), lane, 16 bytes
    __attribute__((aligned(16))) bits16x8 tile[2][S::CT][KS][S::PARTS][WAVE];
    __attribute__((aligned(16))) float nrm[2][S::TC];
    __attribute__((aligned(16))) float ref[16 * KS];  // the reference, scaled
    float cmax[S::NW];
    float spread[S::NW];                              // largest distance of a component from the reference
    int cand[S::TM][6];                               // groups to measure, -1: none; none after the first -1
    float low[4][NB][NT];                             // of the segments before: a thread's smallest minima, ascending,
    int group[3][NB][NT];                             // and the groups of the first three
};

// The cells of up to TM vectors by a workgroup; row(k): the row of x that is vector k, -1 for none.  store(row, cell) for a
// vector that is decided, undecided(row) for one that is not.
template <int NT, int KS, int NB, bool VEC, Factors F, bool PHASES, typename Row, typename Store, typename Undecided>
__device__ __forceinline__ void filter_tile(FilterTile<NT, KS, NB, F> &sh, const float *__restrict__ coarse, int K, int d,
                                            const float *__restrict__ x, int64_t ldx, Row row_of, Store store,
                                            Undecided undecided)
{
    using S = FilterShape<NT, KS, NB, F>;
    constexpr int PS = S::PS, IT = S::IT, NW = S::NW, TC = S::TC, CT = S::CT, TM = S::TM;
    constexpr bool HALF = F == Factors::Half;
    constexpr int D = 16 * KS;
    constexpr int NC = 6;  // groups to measure: three of each lane of a vector
    auto &tile = sh.tile;
    auto &nrm = sh.nrm;
    auto &ref = sh.ref;
    auto &cand = sh.cand;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 31, half = lane >> 5;

    float spread = 0.0f;
    for (int t = tid; t < D; t += NT) {
        ref[t] = reference_component(coarse, K, d, t, &spread);
    }
    if constexpr (HALF) {
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) spread = fmaxf(spread, __shfl_xor(spread, m));
        if (lane == 0) sh.spread[wave] = spread;
    }
    __syncthreads();
    float scale = 1.0f;
    if constexpr (HALF) {
        for (int k = 0; k < NW; ++k) spread = fmaxf(spread, sh.spread[k]);
        if (spread == 0.0f) {  // uniform; those centroids are all the same: the workgroup's first vector then
            const float *xr = x + (int64_t)row_of(0) * ldx;  // (there is a first one)
            for (int t = lane; t < d; t += WAVE) {
                const float f = fabsf(xr[t] - ref[t]);
                if (f < 3e38f) spread = fmaxf(spread, f);
            }
#pragma unroll
            for (int m = 32; m >= 1; m >>= 1) spread = fmaxf(spread, __shfl_xor(spread, m));
        }
        scale = half_scale(spread);
        __syncthreads();  // (nobody still reads the reference as it was)
        for (int t = tid; t < D; t += NT) ref[t] *= scale;
        __syncthreads();
    }

    // this wavefront's vectors: operand -2 x'; lane (col, half) holds components 16 s + 8 half ..
    bits16x8 bh[NB][KS], bl[NB][HALF ? 1 : KS];
    float xn[NB];   // |x'|^2
    float xe2[NB];  // |x' - its operand / -2|^2
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int64_t i = row_of((wave * NB + nb) * 32 + col);
        const float *row = x + (i < 0 ? 0 : i) * ldx;
        float s2 = 0.0f, e2 = 0.0f;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int t = 16 * s + 8 * half;
            f32x8 v = load8<VEC, (KS > 8)>(row, t, d);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                if constexpr (HALF) v[e] = __builtin_fmaf(v[e], scale, -ref[t + e]);  // (zero beyond d)
                else v[e] = v[e] - ref[t + e];
                s2 = __builtin_fmaf(v[e], v[e], s2);
            }
            if constexpr (HALF) {
                const f16x8 h = __builtin_convertvector(v, f16x8);
                const f32x8 err = v - __builtin_convertvector(h, f32x8);
#pragma unroll
                for (int e = 0; e < 8; ++e) e2 = __builtin_fmaf(err[e], err[e], e2);
                bh[nb][s] = __builtin_bit_cast(bits16x8, h * (_Float16)-2.0f);
            } else {
                split_bf16(v * -2.0f, &bh[nb][s], &bl[nb][s]);
            }
        }
        xn[nb] = s2 + __shfl_xor(s2, 32);
        xe2[nb] = e2 + __shfl_xor(e2, 32);
    }

    // Rounding of a score, whatever the unit: |score - (distance^2 - |x'|^2)| <= xerr + cerr, a part of the vector and one
    // of the centroid.  The part of the centroid comes off its score from the start, so that a far centroid loosens its
    // own score and no other's.
    //   Split: both eps |.|^2: the differences 4 2^-24; what the splits and the missing lo.lo leave out 3.1 2^-18; 3 D + 1
    //   additions of values up to 2 (|x'|^2 + |c'|^2) (3 D + 1) 2^-22 (2^-23 each: no assumption on how the matrix units
    //   round); the norms (D + 8) 2^-24; 1.28e-5 + 7.8e-7 D in all.
    //   Half: see qadc_half.h.
    // The number of a group in the low bits of its minimum: log2 (SEG / 8) bits, an error of 2 (SEG / 8) 2^-24 of the score,
    // which is at most |x'|^2 + 2 |c'|^2 (1 + what rounding adds).
    constexpr float eps_g = 1.01f * (float)(S::SEG / 4) / 16777216.0f;
    constexpr float eps = (HALF ? half_eps(D) : 1.5e-5f + 9e-7f * D) + eps_g;
    constexpr float eps_c = (HALF ? half_eps_c(D) : 1.5e-5f + 9e-7f * D) + 2.0f * eps_g;

    // thread -> centroid and steps it converts: eight neighbouring lanes hold eight centroids (their
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
                if (part + PS * it < KS) raw[it][h] = load8<VEC, (KS > 8)>(row, 16 * (part + PS * it) + 8 * h, d);
    };
    float cmax = 0.0f;  // largest |c'|^2
    auto stash = [&](int c0, int buf) {
        float s2 = 0.0f;
        bits16x8 conv[IT][2];
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int s = part + PS * it;
            if (s < KS) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const float4 r0 = *reinterpret_cast<const float4 *>(&ref[16 * s + 8 * h]);
                    const float4 r1 = *reinterpret_cast<const float4 *>(&ref[16 * s + 8 * h + 4]);
                    const f32x8 rv = {r0.x, r0.y, r0.z, r0.w, r1.x, r1.y, r1.z, r1.w};
                    f32x8 v = raw[it][h];
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        if constexpr (HALF) v[e] = __builtin_fmaf(v[e], scale, -rv[e]);
                        else v[e] = v[e] - rv[e];
                        s2 = __builtin_fmaf(v[e], v[e], s2);
                    }
                    if constexpr (HALF) {
                        const f16x8 c = __builtin_convertvector(v, f16x8);
                        conv[it][h] = __builtin_bit_cast(bits16x8, c);
                    } else {
                        bits16x8 hi, lo;
                        split_bf16(v, &hi, &lo);
                        tile[buf][crow >> 5][s][0][h * 32 + (crow & 31)] = hi;
                        tile[buf][crow >> 5][s][S::PARTS - 1][h * 32 + (crow & 31)] = lo;
                    }
                }
            }
        }
#pragma unroll
        for (int m = 8; m < 8 * PS; m <<= 1) s2 += __shfl_xor(s2, m);
        const bool in = c0 + crow < K;
        // (A cell past the last has the last one's components, and 2 x'.c' may be larger than AF_NONE: infinity stays above.)
        const float none = __builtin_inff();
        if (in) cmax = fmaxf(cmax, s2);  // (NaN: left out)
        if constexpr (HALF) {
            // A stray centroid, |c'|^2 > 2^31, may not fit binary16: its score is 0.29 |c'|^2, no more than |c'|^2 - 2 x'.c' of
            // any vector with |x'| <= 2^14.  (One with a NaN: NaN, and no product makes one of the others.)
            const bool stray = !(s2 <= HALF_STRAY);
#pragma unroll
            for (int it = 0; it < IT; ++it)
                if (part + PS * it < KS)
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        tile[buf][crow >> 5][part + PS * it][0][h * 32 + (crow & 31)] = stray ? bits16x8{} : conv[it][h];
            const float own = stray ? 0.29f * s2 : __builtin_fmaf(-eps_c, s2, s2) - HALF_TINY * D;
            nrm[buf][crow] = in ? own : none;  // (its threads all write the same: a branch would part the block of code)
        } else {
            nrm[buf][crow] = in ? s2 * (1.0f - eps_c) : none;
        }
    };

    // 32 cells' scores start at their norms: result r is of cell 8 (r / 4) + 4 half + r % 4 and vector col.
    auto multiply = [&](int buf, int ct, f32x16 (&acc)[NB]) {
        f32x16 init;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const float4 v = *reinterpret_cast<const float4 *>(&nrm[buf][ct * 32 + 8 * g + 4 * half]);
            init[4 * g] = v.x; init[4 * g + 1] = v.y; init[4 * g + 2] = v.z; init[4 * g + 3] = v.w;
        }
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[nb] = init;
        // (in phases the operands of a step are requested two steps ahead: left to itself the compiler requests them where they are used)
        bits16x8 a[3][S::PARTS];
        if constexpr (PHASES) {
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int p = 0; p < S::PARTS; ++p) a[s][p] = tile[buf][ct][s][p][lane];
        }
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            if constexpr (PHASES) {
                if (s + 2 < KS)
#pragma unroll
                    for (int p = 0; p < S::PARTS; ++p) a[(s + 2) % 3][p] = tile[buf][ct][s + 2][p][lane];
                __builtin_amdgcn_sched_barrier(0);
            }
            const bits16x8 ah = PHASES ? a[s % 3][0] : tile[buf][ct][s][0][lane],
                           al = PHASES ? a[s % 3][S::PARTS - 1] : tile[buf][ct][s][S::PARTS - 1][lane];
            if constexpr (HALF) {
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, ah), __builtin_bit_cast(f16x8, bh[nb][s]), acc[nb], 0, 0, 0);
            } else {
                auto bf = [](const bits16x8 &v) { return __builtin_bit_cast(bf16x8, v); };
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf(ah), bf(bh[nb][s]), acc[nb], 0, 0, 0);
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf(al), bf(bh[nb][s]), acc[nb], 0, 0, 0);
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf(ah), bf(bl[nb][HALF ? 0 : s]), acc[nb], 0, 0, 0);
            }
        }
    };
    // A lane's four smallest group minima of the segment, ascending.  A group is four consecutive cells; its number takes the
    // place of the lowest bits of its minimum, so that the two are sorted as one.
    float b1[NB], b2[NB], b3[NB], b4[NB];
    unsigned mask = S::MASK;
    asm("" : "+v"(mask));  // (in a register: one instruction for the exchange of bits)
    auto note = [&](const f32x16 (&acc)[NB], unsigned first) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                float v = fminf(fminf(acc[nb][4 * u], acc[nb][4 * u + 1]), acc[nb][4 * u + 2]);
                v = fminf(fminf(v, acc[nb][4 * u + 3]), AF_NONE);  // (no NaN: the medians would take it for the smallest)
                v = __uint_as_float((__float_as_uint(v) & ~mask) | (PHASES ? first + u : (first + u) & mask));
                b4[nb] = __builtin_amdgcn_fmed3f(b3[nb], b4[nb], v);
                b3[nb] = __builtin_amdgcn_fmed3f(b2[nb], b3[nb], v);
                b2[nb] = __builtin_amdgcn_fmed3f(b1[nb], b2[nb], v);
                b1[nb] = __builtin_amdgcn_fmed3f(b1[nb], v, -AF_NONE);  // (the smaller; a minimum would first make v canonical)
            }
    };
    int a1[NB], a2[NB], a3[NB];  // the groups of b1, b2, b3, once the last segment is done
    fetch(0);
    stash(0, 0);
    if constexpr (!PHASES) fetch(min(TC, K - 1));
    __syncthreads();
    f32x16 acc[2][NB];  // of this 32 cells and of the 32 before, whose minima are taken beside these products
    int buf = 0;
    for (int s0 = 0; s0 < K; s0 += S::SEG) {  // uniform
        const int s1 = min(K, s0 + S::SEG);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            b1[nb] = b2[nb] = b3[nb] = b4[nb] = AF_NONE;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[1][nb][r] = AF_NONE;
        }
        for (int c0 = s0; c0 < s1; c0 += TC, buf ^= 1) {
            if constexpr (PHASES) {
                if (c0 + TC < K) fetch(c0 + TC);  // uniform; travels while this tile is multiplied
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    multiply(buf, ct, acc[0]);
                    note(acc[0], (unsigned)((c0 - s0) / 8 + 4 * ct));
                }
                if (c0 + TC < K) stash(c0 + TC, buf ^ 1);  // uniform; that buffer was read before the last barrier
            } else {
                // one block of code, so that the conversion of the next tile and the minima of the results before are dealt out
                // among the products
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    multiply(buf, ct, acc[ct & 1]);
                    note(acc[(ct & 1) ^ 1], (unsigned)((c0 - s0) / 8 + 4 * ct - 4) & S::MASK);
                    if (ct == 0) {
                        stash(c0 + TC, buf ^ 1);  // (nobody reads what is beyond the last; that buffer was read before the last barrier)
                        fetch(min(c0 + 2 * TC, K - 1));
                    }
                }
                if constexpr (CT == 1) {
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) acc[1][nb] = acc[0][nb];
                }
            }
            __syncthreads();
        }
        if constexpr (!PHASES) note(acc[1], (unsigned)((s1 - s0 - 1) / TC * CT + CT - 1) * 4);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            auto group = [&](float b) { return (int)(__float_as_uint(b) & S::MASK) * 2 + s0 / 4 + half; };
            auto value = [&](float b) { return __uint_as_float(__float_as_uint(b) & ~S::MASK); };
            float v[4] = {value(b1[nb]), value(b2[nb]), value(b3[nb]), value(b4[nb])};
            int g[3] = {group(b1[nb]), group(b2[nb]), group(b3[nb])};
            if (s0 > 0) {  // uniform
                float n[4];
                int h[3];
#pragma unroll
                for (int k = 0; k < 4; ++k) n[k] = sh.low[k][nb][tid];
#pragma unroll
                for (int k = 0; k < 3; ++k) h[k] = sh.group[k][nb][tid];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int gk = g[min(k, 2)];  // (the fourth comes last: all that counts is its value)
                    const bool l1 = v[k] < n[0], l2 = v[k] < n[1], l3 = v[k] < n[2];
                    n[3] = __builtin_amdgcn_fmed3f(n[2], n[3], v[k]);
                    n[2] = __builtin_amdgcn_fmed3f(n[1], n[2], v[k]);
                    n[1] = __builtin_amdgcn_fmed3f(n[0], n[1], v[k]);
                    n[0] = fminf(n[0], v[k]);
                    h[2] = l2 ? h[1] : l3 ? gk : h[2];
                    h[1] = l1 ? h[0] : l2 ? gk : h[1];
                    h[0] = l1 ? gk : h[0];
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) v[k] = n[k];
#pragma unroll
                for (int k = 0; k < 3; ++k) g[k] = h[k];
            }
            if (s1 < K) {  // uniform
#pragma unroll
                for (int k = 0; k < 4; ++k) sh.low[k][nb][tid] = v[k];
#pragma unroll
                for (int k = 0; k < 3; ++k) sh.group[k][nb][tid] = g[k];
            }
            b1[nb] = v[0]; b2[nb] = v[1]; b3[nb] = v[2]; b4[nb] = v[3];
            a1[nb] = g[0]; a2[nb] = g[1]; a3[nb] = g[2];
        }
    }

    // over all the centroids
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) cmax = fmaxf(cmax, __shfl_xor(cmax, m));
    if (lane == 0) sh.cmax[wave] = cmax;
    __syncthreads();
    for (int k = 0; k < NW; ++k) cmax = fmaxf(cmax, sh.cmax[k]);

    // With b1 the smallest score, reached by a cell c*: the closest cell's score is at most b1 + 2 xerr + 2 cerr(c*).
    // |c*'|^2 is at most the largest of all cells, and |c*'| <= |x'| + |x' - c*'| with |x' - c*'|^2 <= b1 + |x'|^2 + what
    // rounding adds: under 1.1 thousandths of |x'|^2 (Split); xerr + 2 cerr(c*) (Half), the latter at most 2.0e-3 |c*'|^2 + a
    // constant, so that |c*'| is at most 1 / (1 - 0.045) of what it is without.  A centroid whose score overflows or is NaN (it
    // loses every comparison) is not the closest to a vector that has one within 1e18 (Split) or within HALF_FAR (Half;
    // nor has a stray one, with 0.29 2^31 at least, reached b1 then).
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int v = (wave * NB + nb) * 32 + col;
        const float low = fminf(b1[nb], __shfl_xor(b1[nb], 32));
        float thr;
        bool sure;  // (comparisons that a NaN fails)
        if constexpr (HALF) {
            const float tiny = HALF_TINY * D;
            const float xerr = __builtin_fmaf(eps, xn[nb], __builtin_fmaf(HALF_CONV, xe2[nb], tiny));
            const float far = 1.05f * (__builtin_sqrtf(xn[nb]) + __builtin_sqrtf(fmaxf(low + xn[nb] + xerr + 2.0f * tiny, 0.0f)));
            const float cn = 1.01f * fminf(far * far, cmax);
            thr = low + 2.001f * (xerr + __builtin_fmaf(eps_c, cn, tiny));
            sure = xn[nb] < HALF_NEAR && low < HALF_FAR && b4[nb] > thr;
        } else {
            const float far = __builtin_sqrtf(xn[nb]) + __builtin_sqrtf(fmaxf(low + xn[nb], 0.0f) + 1.1e-3f * xn[nb]);
            thr = low + 2.0f * __builtin_fmaf(eps, xn[nb], __builtin_fmaf(eps_c, 1.01f * fminf(far * far, cmax), 1e-30f));
            sure = xn[nb] < 1e36f && thr < 1e36f && b4[nb] > thr;
        }
        // this lane's groups in question, then those of the other half; the first entry is never empty
        // unless the vector is left to the kernel after this one
        const int g1 = b1[nb] <= thr ? a1[nb] : -1, g2 = b2[nb] <= thr ? a2[nb] : -1,
                  g3 = b3[nb] <= thr ? a3[nb] : -1;
        const int o1 = __shfl_xor(g1, 32), o2 = __shfl_xor(g2, 32), o3 = __shfl_xor(g3, 32);
        const int other = __shfl_xor((int)sure, 32);  // (asked by all lanes: a lane that does not ask gives nothing)
        const bool all = !(sure && other);
        if (half == 0) {
            // own groups first (they fill up in this order), the others' behind them
            const int k = (g1 >= 0) + (g2 >= 0) + (g3 >= 0);
            int c[NC] = {g1, g2, g3, -1, -1, -1};
#pragma unroll
            for (int e = 0; e < NC; ++e) c[e] = e == k ? o1 : e == k + 1 ? o2 : e == k + 2 ? o3 : c[e];
#pragma unroll
            for (int e = 0; e < NC; ++e) cand[v][e] = all ? -2 : c[e];
            if (all && row_of(v) >= 0) undecided(row_of(v));
        }
    }
    __syncthreads();

    // The groups in question, eight lanes per vector: the four distances of a group in float32, the lanes side by side along
    // the components (a lane per cell would read 64 different lines per load).  A cell that no other comes within the
    // rounding of is the closest; else the cells that do are measured by the definition, a lane each.
    const int r = tid & 7, team = lane & ~7, mine = r >> 1;  // (two lanes end with the same cell, 4 g + mine)
    for (int v = tid >> 3; v < TM; v += NT / 8) {
        const int64_t i = row_of(v);
        if (i < 0 || cand[v][0] < 0) continue;  // uniform over the eight lanes
        const float *xr = x + i * ldx;
        constexpr int W = VEC ? 4 : 1;  // components per load
        float xv[2 * KS];
#pragma unroll
        for (int e = 0; e < 2 * KS / W; ++e)
#pragma unroll
            for (int u = 0; u < W; ++u) {
                const int t = W * (r + 8 * e) + u;
                xv[W * e + u] = VEC || t < d ? xr[t] : 0.0f;
            }
        // distance to cell 4 g + mine
        auto measure = [&](int g) {
            float part[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float *cr = coarse + (size_t)min(4 * g + k, K - 1) * d;
                float acc = 0.0f;
#pragma unroll
                for (int e = 0; e < 2 * KS / W; ++e) {
                    float cv[W];
                    if constexpr (W == 4) {
                        const float4 f = *reinterpret_cast<const float4 *>(cr + 4 * (r + 8 * e));
                        cv[0] = f.x; cv[1] = f.y; cv[2] = f.z; cv[3] = f.w;
                    } else {
                        const int t = r + 8 * e;
                        cv[0] = t < d ? cr[t] : 0.0f;
                    }
#pragma unroll
                    for (int u = 0; u < W; ++u) {
                        const float df = xv[W * e + u] - cv[u];
                        acc = __builtin_fmaf(df, df, acc);
                    }
                }
                part[k] = acc;
            }
            // sums over the eight lanes, halving the cells a lane is responsible for
#pragma unroll
            for (int w = 4; w >= 2; w >>= 1)
#pragma unroll
                for (int k = 0; k < w / 2; ++k) {
                    const bool up = r & w;
                    const float keep = up ? part[k + w / 2] : part[k], give = up ? part[k] : part[k + w / 2];
                    part[k] = keep + __shfl_xor(give, w);
                }
            const float to = part[0] + __shfl_xor(part[0], 1);
            return 4 * g + mine < K && to == to ? to : __builtin_inff();  // (a NaN is never the closest)
        };
        auto lowest = [&](float f) {
#pragma unroll
            for (int w = 4; w >= 2; w >>= 1) f = fminf(f, __shfl_xor(f, w));
            return f;
        };
        // rounding of two sums of d squares (d / 8 + 3 additions, the differences, the squares): (d / 4 + 12) 2^-24,
        // here at least 1.3 times that
        auto slack = [&](float f) { return f + __builtin_fmaf(f, 2e-6f + 3.2e-7f * KS, 1e-33f); };
        auto among = [&](bool near) { return __popcll((__ballot(near) >> team) & 0x55ull); };
        const int g0 = cand[v][0];
        float dist[NC];
        dist[0] = measure(g0);
#pragma unroll
        for (int q = 1; q < NC; ++q) dist[q] = __builtin_inff();
        float close = slack(lowest(dist[0]));
        int rivals = among(dist[0] <= close);
        int bc = dist[0] <= close ? 4 * g0 + mine : 0x7fffffff;
        if (cand[v][1] >= 0) {  // uniform over the eight lanes
            float least = dist[0];
#pragma unroll 1
            for (int q = 1; q < NC; ++q) {
                const int g = cand[v][q];
                if (g < 0) break;  // uniform over the eight lanes
                const float to = measure(g);
                least = fminf(least, to);
#pragma unroll
                for (int p = 1; p < NC; ++p) dist[p] = p == q ? to : dist[p];
            }
            close = slack(lowest(least));
            bc = 0x7fffffff;
            rivals = 0;
#pragma unroll
            for (int q = 0; q < NC; ++q) {
                const bool near = dist[q] <= close && cand[v][q] >= 0;
                rivals += among(near);
                if (near) bc = 4 * cand[v][q] + mine;
            }
        }
        if (rivals > 1) {  // uniform over the eight lanes
            double bd = __builtin_inf();
            bc = 0x7fffffff;
#pragma unroll 1
            for (int q = 0; q < NC; ++q) {
                const int g = cand[v][q];
                float dq = dist[0];
#pragma unroll
                for (int p = 1; p < NC; ++p) dq = p == q ? dist[p] : dq;
                const int c = 4 * g + mine;
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
            for (int w = 4; w >= 2; w >>= 1) {
                const double od = __shfl_xor(bd, w);
                const int oc = __shfl_xor(bc, w);
                if (od < bd || (od == bd && oc < bc)) { bd = od; bc = oc; }
            }
        } else {
#pragma unroll
            for (int w = 4; w >= 2; w >>= 1) bc = min(bc, __shfl_xor(bc, w));
        }
        if (r == 0) store(i, bc);
    }
}

template <int NT, int KS, int NB, bool VEC, Factors F, bool PHASES>
__global__ __launch_bounds__(NT, 2) void assign_filter_kernel(const float *__restrict__ coarse, int K, int d,
                                                              const float *__restrict__ x, int64_t ldx, int64_t n,
                                                              int32_t *__restrict__ cells, int scale, int accumulate)
{
    __shared__ FilterTile<NT, KS, NB, F> sh;
    const int64_t i0 = (int64_t)blockIdx.x * FilterShape<NT, KS, NB, F>::TM;
    filter_tile<NT, KS, NB, VEC, F, PHASES>(
        sh, coarse, K, d, x + i0 * ldx, ldx, [&](int k) { return i0 + k < n ? k : -1; },
        [&](int64_t k, int bc) { cells[i0 + k] = (accumulate ? cells[i0 + k] : 0) + bc * scale; },
        [&](int64_t k) { cells[i0 + k] = (accumulate ? cells[i0 + k] : 0) ^ ASG_MARK; });
}

// ------------------------------------------------------------------ what the filter leaves

// Every workgroup looks for the marks of `range` vectors (a multiple of ASG_TM, up to ASG_RANGE).  More than ASG_FEW of
// them go through the filter again, with split factors, whose margins are a tenth -- until that decides less than a quarter of a
// tile (centroids four times over: 2 ms of 46 wasted on 1 M vectors without this).  Those left it measures
// against all cells, by the definition: 128 at a time in tiles, or, of a few, four at a time and a lane per
// cell (a tile takes as long as five such rounds whatever it holds).  The filter's own last steps were slower at it, and
// cost the filter its registers.  Ranges rather than single tiles, so that few marks fill few tiles; about 1024 workgroups
// (512 at a time: with as many ranges, 200 k vectors that are all marked left a quarter of the chip idle, 1.48 ms).
// AGAIN, DEFINITION: which of the two this launch does (both, but for the 16-step form, which would spill 46 registers:
// 60 against 48 ms for 500 k vectors of 256 components, all marked).
constexpr int ASG_RANGE = 4096, ASG_FEW = 20;

// Copies of a centroid (a list padded to its length, clusters that started from equal vectors, one centroid over and over) leave
// every vector near them to the definition, and add nothing to it: the lowest of equal cells wins.  Before a workgroup measures more
// than a tile of vectors it looks for them, wherever they stand, and lists the other cells, increasing; where there are no copies, or
// more than ASG_LIST other cells, or more than ASG_COPIES_K in all, it returns 0 and nothing is listed.
// Rows are hashed, 16 lanes each; a slot is for the lowest row of a hash, and the others with that hash are compared with it, bit by bit.
// (A copy may go unnoticed where its original found no slot.)  us, with this / all cells measured, 200 k vectors, d = 64, K = 1024:
// one centroid over and over 379 / 1254, the last or the first of them another 309 / 711, two in turn 374 / 1242, 20 of them in any order 373 /
// 1224, 128 eight times each 374 / 1217; K = 4096, d = 128: one 1350 / 9900, 512 eight times 2340 / 9930; K = 16384, d = 32, 30 k
// 2048 eight times 1266 / 2990; no copies 1232 / 1230, 9993 / 10044, 3014 / 3000.
constexpr int ASG_LIST = 4096, ASG_SLOTS = 4096, ASG_COPIES_K = 65536;

struct AssignCopies {
    unsigned long long slots[ASG_SLOTS];  // row << 32 | hash
    unsigned copy[ASG_COPIES_K / 32];     // a bit per row
    unsigned count[4];
    int some;
};

// The sum over the 16 lanes of a row, in all of them.
__device__ __forceinline__ unsigned team_sum(unsigned v)
{
    v += dpp_or_zero<0x128>(v);  // (rotations by 8, 4, 2, 1)
    v += dpp_or_zero<0x124>(v);
    v += dpp_or_zero<0x122>(v);
    return v + dpp_or_zero<0x121>(v);
}

__device__ __forceinline__ int list_cells(AssignCopies &s, uint16_t *list, const float *__restrict__ coarse, int K, int d)
{
    constexpr int U = 8;  // rows of a team (16 lanes) in flight
    constexpr unsigned SLOT = 0x100000000ull / ASG_SLOTS;  // hashes that share a slot
    constexpr int PROBES = 4;
    const int tid = threadIdx.x, r = tid & 15, team = tid >> 4, lane = tid & 63, wave = tid >> 6;
    const unsigned *c = reinterpret_cast<const unsigned *>(coarse);
    for (int i = tid; i < ASG_SLOTS; i += 256) s.slots[i] = ~0ull;
    for (int i = tid; i < (K + 31) / 32; i += 256) s.copy[i] = 0;
    if (tid == 0) s.some = 0;
    __syncthreads();
    auto mix = [](unsigned a) {
        a ^= a >> 16; a *= 0x85ebca6bu;
        a ^= a >> 13; a *= 0xc2b2ae35u;
        return a ^ a >> 16;
    };
    // of row at(c0 + 16 u + team), u = r (r < U): a hash of up to 32 components
    auto hash = [&](int c0, auto at) {
        unsigned h[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const unsigned *row = c + (size_t)at(min(c0 + 16 * u + team, K - 1)) * d;
            unsigned a = 0;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int e = r + 16 * j, t = d > 32 ? e * d >> 5 : e;
                if (t < d) a = (a + row[t]) * 0x9e3779b1u + (unsigned)e;
            }
            h[u] = mix(a);
        }
        unsigned own = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            h[u] = team_sum(h[u]);
            own = r == u ? h[u] : own;
        }
        return mix(own);
    };
    auto insert = [&](int c0, int end, auto at) {
        const unsigned h = hash(c0, at);
        const int k = c0 + 16 * r + team;
        if (r < U && k < end) {
            const int row = at(k);
            const unsigned long long own = (unsigned long long)row << 32 | h;
            for (int p = 0; p < PROBES; ++p) {
                unsigned long long *slot = &s.slots[(h / SLOT + p) % ASG_SLOTS];
                unsigned long long was = atomicCAS(slot, ~0ull, own);
                if (was == ~0ull) break;
                if ((unsigned)was != h) continue;
                was = atomicMin(slot, own);  // (the same hash: the lowest row)
                if (was != own) {
                    const int late = max(row, (int)(was >> 32));
                    atomicOr(&s.copy[late >> 5], 1u << (late & 31));
                    s.some = 1;
                }
                break;
            }
        }
    };
    auto itself = [](int k) { return k; };
    // a sample first: copies that are few are not worth looking for (twice 4096 cells: 8 pairs of the 256 rows)
    const int sample = max(K / 16, 256);
    if (sample < K) {  // uniform
        for (int c0 = 0; c0 < sample; c0 += 16 * U)  // uniform
            insert(c0, sample, [&](int k) { return (int)((uint64_t)mix((unsigned)k + 1u) * (unsigned)K >> 32); });
        __syncthreads();
        if (!s.some) return 0;  // uniform
    }
    for (int c0 = 0; c0 < K; c0 += 16 * U) insert(c0, K, itself);  // uniform
    __syncthreads();
    if (!s.some) return 0;  // uniform
    for (int c0 = 0; c0 < K; c0 += 16 * U) {  // uniform
        const unsigned h = hash(c0, itself);
        const int mine = c0 + 16 * r + team;
        const bool suspect = r < U && mine < K && (s.copy[mine >> 5] >> (mine & 31) & 1u);
        int own = K;
        if (suspect)
            for (int p = 0; p < PROBES && own == K; ++p) {
                const unsigned long long in = s.slots[(h / SLOT + p) % ASG_SLOTS];
                if ((unsigned)in == h && in != ~0ull) own = (int)(in >> 32);
            }
        if (__ballot(suspect) == 0ull) continue;  // uniform over the wavefront
        const unsigned *a[U], *b[U];
        unsigned diff[U] = {};
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int row = min(c0 + 16 * u + team, K - 1), with = __shfl(suspect ? own : mine, (lane & 48) + u);
            a[u] = c + (size_t)row * d;
            b[u] = c + (size_t)min(with, K - 1) * d;
        }
        for (int t = r; t < d; t += 16)
#pragma unroll
            for (int u = 0; u < U; ++u) diff[u] |= a[u][t] ^ b[u][t];
        bool differs = false;  // row r of the team
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool any = team_sum(diff[u] ? 1u : 0u) != 0;
            differs = r == u ? any : differs;
        }
        differs = differs || own >= mine;
        if (suspect && differs) atomicAnd(&s.copy[mine >> 5], ~(1u << (mine & 31)));
    }
    __syncthreads();
    unsigned found = 0;
    for (int c0 = 0; c0 < K; c0 += 256) {  // uniform
        const int row = c0 + tid;
        const bool keep = row < K && !(s.copy[row >> 5] >> (row & 31) & 1u);
        const unsigned long long mask = __ballot(keep);
        if (lane == 0) s.count[wave] = (unsigned)__popcll(mask);
        __syncthreads();
        unsigned at = found + rank_in_mask(mask);
        for (int w = 0; w < 4; ++w) {
            if (w < wave) at += s.count[w];
            found += s.count[w];
        }
        if (keep && at < (unsigned)ASG_LIST) list[at] = (uint16_t)row;
        __syncthreads();
    }
    return found <= (unsigned)ASG_LIST ? (int)found : 0;
}

template <int KS, bool VEC, bool AGAIN, bool DEFINITION>
__global__ __launch_bounds__(256) void assign_rest_kernel(const float *__restrict__ coarse, int K, int d,
                                                          const float *__restrict__ x, int64_t ldx, int64_t n, int range,
                                                          int32_t *__restrict__ cells, int scale, int accumulate)
{
    using Again = FilterTile<256, KS, 1, Factors::Split>;
    constexpr int TM = FilterShape<256, KS, 1, Factors::Split>::TM;
    constexpr size_t BYTES = DEFINITION && (!AGAIN || sizeof(AssignTile) > sizeof(Again)) ? sizeof(AssignTile) : sizeof(Again);
    static_assert(sizeof(AssignCopies) <= sizeof(AssignTile), "");
    __shared__ __attribute__((aligned(16))) char room[BYTES];  // for one of them at a time
    AssignTile &s = *reinterpret_cast<AssignTile *>(room);
    __shared__ uint16_t todo[ASG_RANGE];
    __shared__ uint16_t list[DEFINITION ? ASG_LIST : 1];
    __shared__ int ntodo, nleft;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t i0 = (int64_t)blockIdx.x * range;
    if (tid == 0) { ntodo = 0; nleft = 0; }
    __syncthreads();
    for (int k = tid; k < range; k += 256) {
        const bool found = i0 + k < n && assign_marked(cells[i0 + k], K, accumulate);
        if (found) todo[atomicAdd(&ntodo, 1)] = (uint16_t)k;
    }
    __syncthreads();
    int count = ntodo;
    if (count == 0) return;  // uniform
    if constexpr (AGAIN) {
        if (count > ASG_FEW) {  // uniform
            int behind = 0;  // undecided in the tiles so far
            for (int k0 = 0; k0 < count; k0 += TM) {  // uniform
                filter_tile<256, KS, 1, VEC, Factors::Split, true>(
                    *reinterpret_cast<Again *>(room), coarse, K, d, x + i0 * ldx, ldx,
                    [&](int k) { return k0 + k < count ? (int)todo[k0 + k] : -1; },
                    [&](int64_t k, int bc) { cells[i0 + k] = (cells[i0 + k] ^ ASG_MARK) + bc * scale; },
                    [&](int64_t) { atomicAdd(&nleft, 1); });
                __syncthreads();
                const int left = nleft;
                if (4 * (left - behind) > 3 * min(TM, count - k0)) break;  // uniform
                behind = left;
                __syncthreads();
            }
            // the vectors still marked (a thread sees the cells it looks at as the workgroup has left them: behind a barrier)
            __threadfence_block();
            __syncthreads();
            if (tid == 0) nleft = 0;
            __syncthreads();
            for (int c0 = 0; c0 < count; c0 += 256) {  // uniform; the list shrinks in place
                const int k = c0 + tid < count ? todo[c0 + tid] : -1;
                __syncthreads();
                if (k >= 0 && assign_marked(cells[i0 + k], K, accumulate)) todo[atomicAdd(&nleft, 1)] = (uint16_t)k;
                __syncthreads();
            }
            count = nleft;
        }
    }
    if constexpr (!DEFINITION) return;
    auto store = [&](int k, int bc) { cells[i0 + k] = (cells[i0 + k] ^ ASG_MARK) + bc * scale; };
    const int few = d <= 4 ? ASG_RANGE : ASG_FEW;  // (a tile computes 16 components at least)
    int k0 = 0, listed = 0;
    if (count > min(few, ASG_TM) && K <= ASG_COPIES_K) {  // uniform
        listed = list_cells(*reinterpret_cast<AssignCopies *>(room), list, coarse, K, d);
        if (listed) K = listed;
        __syncthreads();
    }
    auto cell = [&](int k) { return listed ? (int)list[k] : k; };
    for (; count - k0 > few; k0 += ASG_TM) {  // uniform
        assign_tile(s, coarse, K, d, x + i0 * ldx, ldx, [&](int k) { return k0 + k < count ? (int)todo[k0 + k] : -1; }, cell, store);
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
            const float *cr = coarse + (size_t)cell(c) * d;
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
            store(todo[k0 + tid], c0 == 0x7fffffff ? c0 : cell(c0));
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------------ host

// One binary16 product per component, or factors split into two bfloat16 numbers from the start?  The first leaves more
// vectors undecided, for which the split form and the float64 tiles come after it.  Its time over that of the split form, vectors
// well inside their cells / vectors and centroids of one Gaussian, where most vectors have rivals: 1 M vectors, d = 128, K = 4096
// 0.51 / 0.56, d = 32, K = 1024 0.76 / 0.90, 120 k d = 256, K = 16384 0.74 / 0.90, 60 k d = 64, K = 4096 0.67 / 1.18, d = 128,
// K = 256 0.95 / 1.15; but where a call is less than a round of workgroups (10 k, K = 4096, d = 64 0.87 / 1.56, d = 96 0.87 / 1.43;
// 30 k, d = 128, K = 256 0.96 / 1.02; 60 k, d = 32, K = 16384 0.72 / 1.12), in few dimensions (1 M, d = 2, K = 4096 1.66, d = 16,
// K = 64 0.97 / 1.09, d = 24, K = 256 0.93 / 1.08) and for rows that are not whole steps (1 M, d = 100, K = 64 0.98 / 1.08,
// d = 200, K = 256 0.93 / 1.13) a tenth is won where all is well and more lost where it is not.
static bool half_factors_pay(int K, int d, int64_t n, bool vec)
{
    if (vec && n >= 49152 && (d >= 64 ? K >= 256 : K >= 1024 && K <= 4096)) return true;
    if (n < 98304 || (d > 128 && !vec)) return false;
    if (vec || (d > 32 && d <= 64)) return true;
    return d >= 8 && K >= (d > 64 ? 1024 : 4096);
}

// 512 (256 beyond 128 components) vectors per workgroup, or 128?  The wide form converts the centroids a quarter as often and is
// one workgroup per compute unit; it loses where the chip is not filled and the walk over the centroids is short.  us, narrow /
// wide: K = 4096, d = 128 50 k 129 / 112, 66 k 190 / 113, 131 k 312 / 149, 262 k 512 / 288; d = 64 50 k 69 / 74, 66 k 102 / 76,
// 148 k 194 / 157; d = 256 50 k 251 / 179, 262 k 1017 / 751; d = 32 66 k 62 / 61, 115 k 83 / 62, 148 k 103 / 118, 197 k 132 / 118;
// K = 256, d = 128 66 k 35 / 35, 115 k 49 / 37, 148 k 56 / 65, 197 k 73 / 68, 262 k 83 / 72; d = 64 115 k 26 / 25, 148 k 34 / 44,
// 262 k 47 / 48; d = 256 66 k 68 / 74, 115 k 83 / 77, 262 k 160 / 152.
template <int KS>
static bool wide_pays(int K, int64_t n)
{
    if (K >= 1024 && KS > 2) return n >= (KS > 8 ? 32768 : 65536);
    if (KS > 8) return n >= 98304;
    const int64_t round = 512 * 256;  // vectors that fill the chip once
    if (K >= 1024 || KS > 4) return n >= 3 * round / 4 && (n <= round || n >= 3 * round / 2);
    return n >= 2 * round;
}

// Split factors: the minima and the conversion of the centroids in one block of code with the products, or in phases of their own,
// the operands of a product requested two steps ahead?  The block is for wavefronts that are alone on a SIMD; two of them have
// each other's products to run beside, up to 128 components, and 16 steps of products leave no registers for it.  Rows that are not
// whole steps are converted behind a branch per load, which parts the block: phases from 65 components on.  us, block / phases (before
// there was a block), K = 16384: d = 128 20 k 536 / 579 (576), 40 k 702 / 632 (625); d = 64 20 k 267 / 302 (291), 40 k 360 / 342
// (329); d = 256 20 k 955 / 892 (910), 40 k 1247 / 1118 (1139); d = 100 20 k 905 / 816 (821); d = 200 100 k 3024 / 2752 (2900); d = 63
// 40 k 434 / 472 (466); K = 1000: d = 128 20 k 42.6 / 45.5 (54.0), 40 k 58.9 / 55.5 (66.6); d = 256 20 k 76.6 / 71.7 (86.4).
template <int KS, bool VEC>
static bool phases_pay(int64_t n)
{
    return VEC ? KS > 8 || n > 128 * 256 : KS > 4;
}

template <int KS>
static void launch_filter(const float *coarse, int K, int d, const float *x, int64_t ldx, int64_t n, int range,
                          int32_t *cells, int scale, int accumulate, hipStream_t st)
{
    const bool vec = d == 16 * KS && ldx % 4 == 0 && ((uintptr_t)coarse & 15) == 0 && ((uintptr_t)x & 15) == 0;
    const dim3 grid((unsigned)ceil_div(n, 128)), ranges((unsigned)ceil_div(n, range));
#define QADC_FILTER(NT_, NB_, VEC_, F_, PHASES_, GRID_)                                                                    \
    hipLaunchKernelGGL((assign_filter_kernel<NT_, KS, NB_, VEC_, Factors::F_, PHASES_>), GRID_, dim3(NT_), 0, st, coarse,  \
                       K, d, x, ldx, n, cells, scale, accumulate)
#define QADC_REST(VEC_, AGAIN_, DEFINITION_)                                                                               \
    hipLaunchKernelGGL((assign_rest_kernel<AGAIN_ ? KS : 2, VEC_, AGAIN_, DEFINITION_>), ranges, dim3(256), 0, st, coarse, K, \
                       d, x, ldx, n, range, cells, scale, accumulate)
    constexpr bool ONE = KS <= 8;
    if (!half_factors_pay(K, d, n, vec)) {
        if (vec) {
            if (phases_pay<KS, true>(n)) QADC_FILTER(256, 1, true, Split, true, grid);
            else if constexpr (KS <= 8) QADC_FILTER(256, 1, true, Split, false, grid);
        } else {
            if (phases_pay<KS, false>(n)) {
                if constexpr (KS > 4) QADC_FILTER(256, 1, false, Split, true, grid);
            } else if constexpr (KS <= 4) {
                QADC_FILTER(256, 1, false, Split, false, grid);
            }
        }
        QADC_REST(false, false, true);
        return;
    }
    if (vec) {
        const bool wide = wide_pays<KS>(K, n);
        if (wide) {
            if constexpr (KS <= 8) QADC_FILTER(512, 2, true, Half, false, dim3((unsigned)ceil_div(n, 512)));
            else QADC_FILTER(512, 1, true, Half, false, dim3((unsigned)ceil_div(n, 256)));
        }
        if (!wide) QADC_FILTER(256, 1, true, Half, false, grid);
        QADC_REST(true, true, ONE);
    } else {
        if constexpr (KS <= 8) {  // (half_factors_pay: no more components)
            // (rows that are not whole steps: us, narrow / wide (groups of 16 cells, narrow), 100 k vectors, K = 16384: d = 40 441 / 311
            // (392), d = 63 615 / 325 (618), d = 80 847 / 530 (1380); K = 4096: d = 40 123 / 90 (127); 148 k 188 / 177 (206), vectors
            // and centroids of one Gaussian 228 / 232 (266); K = 2048 134 / 150 (172))
            bool wide = false;
            if constexpr (KS == 4 || KS == 6) {
                wide = K >= 4096;
                if (wide) QADC_FILTER(512, 2, false, Half, false, dim3((unsigned)ceil_div(n, 512)));
            }
            if (!wide) QADC_FILTER(256, 1, false, Half, false, grid);
            QADC_REST(false, true, ONE);
        }
    }
    if constexpr (!ONE) QADC_REST(false, false, true);
#undef QADC_FILTER
#undef QADC_REST
}

// cells[i] = (accumulate ? cells[i] : 0) + scale * (closest of K centroids to the d components at x + i ldx)
static int assign_pass(const float *coarse, int K, int d, const float *x, int64_t ldx, int64_t n, int32_t *cells,
                       int scale, int accumulate, hipStream_t st)
{
    const bool filter = d <= AF_MAX_D && K <= ASG_MARK_MAX_K;
    const int range = (int)std::min<int64_t>(ASG_RANGE, std::max<int64_t>(256, ceil_div(ceil_div(n, 1024), ASG_TM) * ASG_TM));
    if (!filter)
        hipLaunchKernelGGL(assign_f64_kernel, dim3((unsigned)ceil_div(n, ASG_TM)), dim3(256), 0, st, coarse, K, d, x,
                           ldx, n, cells, scale, accumulate);
    else if (d <= 32)
        launch_filter<2>(coarse, K, d, x, ldx, n, range, cells, scale, accumulate, st);
    else if (d <= 64)
        launch_filter<4>(coarse, K, d, x, ldx, n, range, cells, scale, accumulate, st);
    else if (d <= 96)
        launch_filter<6>(coarse, K, d, x, ldx, n, range, cells, scale, accumulate, st);
    else if (d <= 128)
        launch_filter<8>(coarse, K, d, x, ldx, n, range, cells, scale, accumulate, st);
    else
        launch_filter<16>(coarse, K, d, x, ldx, n, range, cells, scale, accumulate, st);
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
