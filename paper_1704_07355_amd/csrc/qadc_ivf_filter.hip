// Index step of large calls (Section 2.2 of the paper) on the matrix units: for every query and every group of four
// cells, a lower bound of the smallest distance, from binary16 factors (qadc_half.h).  ivf_select_filtered_kernel takes the
// groups that can hold one of the nprobe closest cells from them and measures those cells by the definition, so the cells
// chosen are the definition's; a query the bounds cannot serve is left to the kernels of the float32 distances.
//
// Bound by latency: wavefronts (two per SIMD at 1024 queries x 65536 cells) wait for two thirds of their cycles, the matrix units
// are busy a fifth; the bounds, 8 bytes per lane, tile and query, leave the L2 in parts of lines (98 MB for 33).  4096
// queries x 65536 cells of 128 components (four launches): 185 us, 15 for the factors and 283 for the
// selection, where the float32 distances of all pairs took 1590 and 80; 1000 x 16384 10 + 7 + 58.  (Tiles of cells from memory
// straight into registers, a tile ahead: 348 us, 26 registers spilled.)
#include <algorithm>

#include "qadc_common.h"
#include "qadc_half.h"
#include "qadc_ivf_filter.h"
#include "qadc_profile.h"

namespace qadc {

constexpr int IVFF_MAX_D = 256;

// The bounds are of exact distances, the definition is the float32 one: they order cells alike where its squares neither overflow
// nor lose bits below the normal range, that is for scales (half_scale) within these.  A square that matters is at most
// 4 HALF_FAR / scale^2 < 2^124; what a sum of D squares loses below 2^-126, at most D 2^-150 scale^2 of the scaled one, is far
// inside HALF_TINY D.  Outside (centroids less than 3e-11 or more than 2e15 apart) every query is left to the float32 distances,
// whose ties the bounds would break.
constexpr float IVFF_MIN_SCALE = 0x1p-46f, IVFF_MAX_SCALE = 0x1p+39f;

// Tiles of 32 rows as the matrix instructions read them: step s of 16 components, lane (row, half), 16 bytes.  Workgroup b <
// ctiles takes centroids: operand c^ and the lower bound of |c'|^2 for the scores (minus infinity for a centroid with a
// NaN: no query can then rely on the bounds).  The others take queries: operand -2 x^, and (|x'|^2, ex^2), NaN where the
// bounds are not to be used.
template <int KS>
__global__ __launch_bounds__(256) void ivf_filter_convert_kernel(const float *__restrict__ coarse, int K, int d,
                                                                 const float *__restrict__ queries, int nq, int ctiles,
                                                                 int vec, bits16x8 *__restrict__ cells,
                                                                 float *__restrict__ nrm, bits16x8 *__restrict__ qs,
                                                                 float2 *__restrict__ qstat)
{
    constexpr int D = 16 * KS;
    __shared__ __attribute__((aligned(16))) float ref[D];
    __shared__ float spread_s[256 / WAVE];
    const int tid = threadIdx.x, lane = lane_id();
    float spread = 0.0f;
    for (int t = tid; t < D; t += 256) ref[t] = reference_component(coarse, K, d, t, &spread);
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) spread = fmaxf(spread, __shfl_xor(spread, m));
    if (lane == 0) spread_s[tid / WAVE] = spread;
    __syncthreads();
    for (int k = 0; k < 256 / WAVE; ++k) spread = fmaxf(spread, spread_s[k]);
    if (spread == 0.0f) {  // uniform; those centroids are all the same: the first query then
        for (int t = lane; t < d; t += WAVE) {
            const float f = fabsf(queries[t] - ref[t]);
            if (f < 3e38f) spread = fmaxf(spread, f);
        }
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) spread = fmaxf(spread, __shfl_xor(spread, m));
    }
    const float scale = half_scale(spread);

    const bool is_cell = (int)blockIdx.x < ctiles;  // uniform
    const int tile = is_cell ? (int)blockIdx.x : (int)blockIdx.x - ctiles;
    const int r = tid >> 3, part = tid & 7;
    const int row = tile * 32 + r, rows = is_cell ? K : nq;
    const bool in = row < rows;
    const float *src = (is_cell ? coarse : queries) + (size_t)min(row, rows - 1) * d;
    bits16x8 *dst = (is_cell ? cells : qs) + (size_t)tile * KS * WAVE;
    constexpr int IT = (KS + 7) / 8;
    float s2 = 0.0f, e2 = 0.0f;
    bits16x8 conv[IT][2];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const int s = part + 8 * it;
        if (s < KS) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int t = 16 * s + 8 * h;
                f32x8 v = vec && t + 8 <= d ? load8<true>(src, t, d) : load8<false>(src, t, d);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    v[e] = __builtin_fmaf(v[e], scale, -(ref[t + e] * scale));  // (zero beyond d)
                    s2 = __builtin_fmaf(v[e], v[e], s2);
                }
                const f16x8 c = __builtin_convertvector(v, f16x8);
                const f32x8 err = v - __builtin_convertvector(c, f32x8);
#pragma unroll
                for (int e = 0; e < 8; ++e) e2 = __builtin_fmaf(err[e], err[e], e2);
                conv[it][h] = __builtin_bit_cast(bits16x8, is_cell ? c : c * (_Float16)-2.0f);
            }
        }
    }
#pragma unroll
    for (int m = 1; m < 8; m <<= 1) {
        s2 += __shfl_xor(s2, m);
        e2 += __shfl_xor(e2, m);
    }
    const bool zero = !in || (is_cell && !(s2 <= HALF_STRAY));
#pragma unroll
    for (int it = 0; it < IT; ++it)
        if (part + 8 * it < KS)
#pragma unroll
            for (int h = 0; h < 2; ++h) dst[(part + 8 * it) * WAVE + h * 32 + r] = zero ? bits16x8{} : conv[it][h];
    if (part != 0) return;
    if (is_cell) {
        float own = s2 <= HALF_STRAY ? __builtin_fmaf(-half_eps_c(D), s2, s2) - HALF_TINY * D : 0.29f * s2;
        if (!(s2 == s2)) own = -__builtin_inff();
        nrm[row] = in ? own : __builtin_inff();  // (rows are padded to whole tiles)
    } else if (in) {
        const bool usable = scale >= IVFF_MIN_SCALE && scale <= IVFF_MAX_SCALE;
        qstat[row] = make_float2(usable ? s2 : __builtin_nanf(""), e2);
    }
}

// A wavefront holds the operands of 32 NBQ queries in registers; the tiles of cells pass through LDS, STAGE at a time, the
// next ones on their way there (without a register) while these are multiplied.  wq: wavefronts of a workgroup side by side
// along the queries; the 4 / wq along the cells share out the tiles of a stage.  Result (cell 8 g + 4 half + k, query) of a tile:
// the smallest of k = 0 .. 3, plus |x'|^2, as bfloat16 at its place in the query's row (qadc_ivf_filter.h).
template <int KS>
struct FilterRoom {
    static constexpr int NBQ = KS <= 8 ? 4 : 2;
    static constexpr int STAGE = KS <= 8 ? 4 : 2;
    __attribute__((aligned(16))) bits16x8 cells[2][STAGE][KS][WAVE];
    __attribute__((aligned(16))) float nrm[2][STAGE * 32];
};

// Lane l: 16 (4) bytes from its address to `to` + 16 l (4 l).
typedef const __attribute__((address_space(1))) unsigned *global_words;
typedef __attribute__((address_space(3))) unsigned *lds_words;
__device__ __forceinline__ void load16_to_lds(const void *from, void *to)
{
    __builtin_amdgcn_global_load_lds((global_words)(uintptr_t)from, (lds_words)to, 16, 0, 0);
}
__device__ __forceinline__ void load4_to_lds(const void *from, void *to)
{
    __builtin_amdgcn_global_load_lds((global_words)(uintptr_t)from, (lds_words)to, 4, 0, 0);
}

template <int KS>
__global__ __launch_bounds__(256, 2) void ivf_filter_kernel(const bits16x8 *__restrict__ cells, const float *__restrict__ nrm,
                                                            int K, const bits16x8 *__restrict__ qs,
                                                            const float2 *__restrict__ qstat, int nq, int wq,
                                                            int per_block, float *__restrict__ dist,
                                                            unsigned *__restrict__ rest)
{
    using Room = FilterRoom<KS>;
    constexpr int NBQ = Room::NBQ, STAGE = Room::STAGE;
    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    __shared__ Room sh;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = lane & 31, half = lane >> 5;
    const int tiles = (K + 31) / 32;
    const int q0 = ((int)blockIdx.y * wq + wave % wq) * 32 * NBQ;
    const int t0 = (int)blockIdx.x * per_block, t1 = min(tiles, t0 + per_block);
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *rest = 0;  // ivf_select_filtered_kernel counts in it
    if (t0 >= t1) return;  // uniform
    auto stage = [&](int t, int buf) {  // (tiles beyond the last: the last one again)
#pragma unroll
        for (int i = 0; i < STAGE * KS / 4; ++i) {
            const int e = 4 * i + wave, tile = min(t + e / KS, tiles - 1);
            load16_to_lds(cells + ((size_t)tile * KS + e % KS) * WAVE + lane, &sh.cells[buf][e / KS][e % KS][0]);
        }
        if (wave < STAGE / 2)
            load4_to_lds(nrm + (size_t)min(t + 2 * wave + half, tiles - 1) * 32 + col, &sh.nrm[buf][wave * WAVE]);
    };
    stage(t0, 0);
    bits16x8 b[NBQ][KS];
    float xn[NBQ];
    uint16_t *out[NBQ];
#pragma unroll
    for (int nb = 0; nb < NBQ; ++nb) {
        // (blocks of queries that do not exist: the last one again, never stored)
        const int qt = min(q0 / 32 + nb, (nq - 1) / 32);
        const int q = min(q0 + 32 * nb + col, nq - 1);
#pragma unroll
        for (int s = 0; s < KS; ++s) b[nb][s] = qs[((size_t)qt * KS + s) * WAVE + lane];
        xn[nb] = qstat[q].x;
        out[nb] = ivf_filter_row(dist, K, (size_t)q) + ivf_filter_place(0, half, 0);
    }
    __syncthreads();
    int buf = 0;
    for (int t = t0; t < t1; t += STAGE, buf ^= 1) {  // uniform
        if (t + STAGE < t1) stage(t + STAGE, buf ^ 1);  // (read before the last barrier)
        if (q0 < nq) {
#pragma unroll 1
            for (int k = wave / wq; k < STAGE; k += 4 / wq) {
                if (t + k >= t1) break;
                f32x16 start;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const f32x4 v = *reinterpret_cast<const f32x4 *>(&sh.nrm[buf][k * 32 + 8 * g + 4 * half]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) start[4 * g + e] = v[e];
                }
#pragma unroll
                for (int n0 = 0; n0 < NBQ; n0 += 2) {  // two independent chains of products
                    f32x16 acc[2] = {start, start};
#pragma unroll
                    for (int s = 0; s < KS; ++s) {
                        const f16x8 a = __builtin_bit_cast(f16x8, sh.cells[buf][k][s][lane]);
#pragma unroll
                        for (int e = 0; e < 2; ++e)
                            acc[e] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, __builtin_bit_cast(f16x8, b[n0 + e][s]), acc[e], 0, 0, 0);
                    }
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const int nb = n0 + e;
                        f32x4 v;
#pragma unroll
                        for (int g = 0; g < 4; ++g)
                            v[g] = fminf(fminf(acc[e][4 * g], acc[e][4 * g + 1]), fminf(acc[e][4 * g + 2], acc[e][4 * g + 3])) + xn[nb];
                        if (q0 + 32 * nb + col < nq)
                            *reinterpret_cast<bf16x4 *>(out[nb] + ivf_filter_place(t + k, 0, 0)) = __builtin_convertvector(v, bf16x4);
                    }
                }
            }
        }
        __syncthreads();
    }
}

// Bytes that ivf_filter needs for nq queries and K centroids of d components, beside a row of K floats per query.
size_t ivf_filter_bytes(int K, int d, int nq)
{
    const int64_t ks = ceil_div(d, 16) <= 2 ? 2 : ceil_div(d, 16) <= 4 ? 4 : ceil_div(d, 16) <= 6 ? 6 : ceil_div(d, 16) <= 8 ? 8 : 16;
    const int64_t ct = ceil_div(K, 32), qt = ceil_div(nq, 32);
    return (size_t)((ct + qt) * ks * 1024 + ct * 128) + align_up((size_t)nq * 12 + 4, 256);
}

// Worth its launches and a longer selection?  Whole calls over 2e5 codes, cells and queries of a mixture, all launches included,
// against the float32 distances of every pair: at 2.5e8 to 7e8 products (queries x cells x components) 0.80 to 0.98 of the time where
// the cells are 128 times the probes and more (d = 32, 2500 queries, K = 8192, 64 probes 1.03), from 1e9 on 0.5 to 0.95; at 1e8
// to 2.5e8 0.87 to 1.01; below, and at 64 cells a probe -- too many groups are as close -- up to 1.12; K = 2048 0.86 to 1.06.
// Calls of up to 32 queries have kernels of their own.
bool ivf_filter_pays(int K, int d, int nq, int nprobe)
{
    return d <= IVFF_MAX_D && nq > 32 && K >= 4096 && K >= 128 * nprobe && (double)nq * K * d >= 2.5e8;
}

struct IvfFilter {
    bits16x8 *cells, *qs;
    float *nrm;
    float2 *qstat;
    unsigned *rest;
};

static IvfFilter filter_parts(void *room, int K, int d, int nq, int ks)
{
    const size_t ct = (size_t)ceil_div(K, 32), qt = (size_t)ceil_div(nq, 32);
    char *p = (char *)room;
    IvfFilter f;
    f.cells = (bits16x8 *)p;
    f.qs = (bits16x8 *)(p + ct * ks * 1024);
    f.nrm = (float *)(p + (ct + qt) * ks * 1024);
    f.qstat = (float2 *)(p + (ct + qt) * ks * 1024 + ct * 128);
    f.rest = (unsigned *)(f.qstat + nq);
    return f;
}

template <int KS>
static void convert(const float *coarse, int K, int d, const float *queries, int nq, void *room, hipStream_t st)
{
    const IvfFilter f = filter_parts(room, K, d, nq, KS);
    const int vec = d % 4 == 0 && ((uintptr_t)coarse & 15) == 0 && ((uintptr_t)queries & 15) == 0;
    const int ct = (int)ceil_div(K, 32), qt = (int)ceil_div(nq, 32);
    launch(QADC_PROF_IVF_INDEX, ivf_filter_convert_kernel<KS>, dim3((unsigned)(ct + qt)), dim3(256), 0, st, coarse, K, d,
           queries, nq, ct, vec, f.cells, f.nrm, f.qs, f.qstat);
}

template <int KS>
static const float2 *filter(int K, int d, int nq, int i0, int ni, void *room, float *dist, unsigned **rest, hipStream_t st)
{
    constexpr int NBQ = FilterRoom<KS>::NBQ, STAGE = FilterRoom<KS>::STAGE;
    const IvfFilter f = filter_parts(room, K, d, nq, KS);
    const int tiles = (int)ceil_div(K, 32), sets = (int)ceil_div(ni, 32 * NBQ);
    const int wq = sets >= 4 ? 4 : sets >= 2 || STAGE < 4 ? 2 : 1;
    // two workgroups per compute unit
    const int rows = (int)ceil_div(sets, wq);
    const int per_block = (int)ceil_div(std::max<int64_t>(1, ceil_div((int64_t)tiles * rows, 512)), STAGE) * STAGE;
    launch(QADC_PROF_IVF_INDEX, ivf_filter_kernel<KS>, dim3((unsigned)ceil_div(tiles, per_block), (unsigned)rows), dim3(256), 0, st,
           (const bits16x8 *)f.cells, (const float *)f.nrm, K, (const bits16x8 *)(f.qs + (size_t)(i0 / 32) * KS * WAVE),
           (const float2 *)(f.qstat + i0), ni, wq, per_block, dist, f.rest);
    *rest = f.rest;
    return f.qstat + i0;
}

#define QADC_FILTER_CASES(CALL_)              \
    if (d <= 32) { CALL_(2); }                \
    else if (d <= 64) { CALL_(4); }           \
    else if (d <= 96) { CALL_(6); }           \
    else if (d <= 128) { CALL_(8); }          \
    else { CALL_(16); }

// The factors of all centroids and of nq queries, in `room` (ivf_filter_bytes).
void ivf_filter_convert(const float *coarse, int K, int d, const float *queries, int nq, void *room, hipStream_t st)
{
#define QADC_CALL(KS_) convert<KS_>(coarse, K, d, queries, nq, room, st)
    QADC_FILTER_CASES(QADC_CALL)
#undef QADC_CALL
}

// The bounds of queries i0 .. i0 + ni - 1 (i0 a multiple of 32) in the rows of `dist`; returns their (|x'|^2, ex^2), the
// number of components the rounding is bounded for, and a counter (zero after the kernel) with room for nq numbers behind it.
const float2 *ivf_filter(int K, int d, int nq, int i0, int ni, void *room, float *dist, int *components, unsigned **rest,
                         hipStream_t st)
{
    const float2 *r = nullptr;
#define QADC_CALL(KS_) r = filter<KS_>(K, d, nq, i0, ni, room, dist, rest, st), *components = 16 * KS_
    QADC_FILTER_CASES(QADC_CALL)
#undef QADC_CALL
    return r;
}

}  // namespace qadc
