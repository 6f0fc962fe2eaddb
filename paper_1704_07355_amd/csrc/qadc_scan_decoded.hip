// Quick ADC scan (Alg. 2 of the paper) of query batches by products of decoded codes (qadc_decoded.h): scan_u8_mfma_kernel's
// work with half of its matrix instructions and a quarter of its table operands, for 4-bit codes whose sub-vectors have up to
// four components, where the codebooks and the queries are at hand (qadc_search).
//
// Bound: instruction issue.  A block of 32 codes x 32 queries takes a SIMD 303 cycles (16-byte codes): 128 of them in the matrix unit
// (42 % busy; 38 % over all four parts), with 32 vector, 7.5 LDS and 5.7 scalar instructions beside its products (lookups of decoded
// components, tests of results); either of the two wavefronts that 214 registers leave (three for 8-byte codes: 156) issues in 43 % of its cycles
// and waits to issue in 33 %.  100 M codes of 16 bytes x 256 queries, a mixture's vectors: the whole search 5.31 ms with
// scan_u8_mfma_kernel, 4.00 here (4e-3 of the pairs pass the first part, 4e-4 the last); 73 M codes of 8 bytes x 256 queries 2.12 -> 1.46.

#include <algorithm>
#include <type_traits>

#include "qadc_scan_common.h"
#include "qadc_scan_tiled.h"
#include "qadc_decoded.h"

namespace qadc {

// Operands of a batch, a workgroup per query and a thread per (table, centroid): the decoded tables (the same from every
// workgroup; the first one writes them), the query's int8 components negated, S and the floor of sum a_j / 4.
template <int B>
__global__ __launch_bounds__(32 * B) void decoded_prepare_kernel(const float *__restrict__ codebooks, int d,
                                                                 const float *__restrict__ queries,
                                                                 const uint8_t *__restrict__ qluts,
                                                                 const float *__restrict__ deltas, int nbins,
                                                                 int *__restrict__ tables, int *__restrict__ operands,
                                                                 int2 *__restrict__ scales, unsigned *__restrict__ left,
                                                                 int left_words)
{
    constexpr int m = 2 * B, NT = 32 * B;
    __shared__ float wmax[NT / WAVE];
    __shared__ int total, none;
    const int tid = threadIdx.x, q = blockIdx.x;
    const int j = tid >> 4, c = tid & 15, dsub = d / m;
    float cv[4], mid[4], yv[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        cv[t] = t < dsub ? codebooks[(size_t)tid * dsub + t] : 0.0f;
        yv[t] = t < dsub ? queries[(size_t)q * d + j * dsub + t] : 0.0f;
    }
    const int e = qluts[(size_t)q * (m * 16) + tid];
    const float delta = deltas[q];
    if (tid == 0) total = none = 0;
    const float s = decoded_scale<NT>(cv, mid, wmax);  // (a barrier inside)
    const int S = decoded_steps(delta, s);
    int phi, yhat;
    const int a = decoded_slack(cv, mid, yv, s, S, e, nbins, &phi, &yhat);
    if (q == 0) tables[tid] = phi;
    for (int i = q * NT + tid; i < left_words; i += gridDim.x * NT) left[i] = 0;
    if (c == 0) {
        operands[(size_t)q * m + ((j >> 3) * 2 + (j & 1)) * 4 + ((j >> 1) & 3)] = yhat;
        if (a == INT32_MAX) none = 1;
        else atomicAdd(&total, a);
    }
    __syncthreads();
    if (tid == 0) scales[q] = none ? make_int2(-1, 0) : make_int2(S, total >> 2);
}

// A wavefront scans units of the database for 32 G queries: per 32 codes it looks up the decoded components of the 32 codes
// once, and 32 G queries' products follow (a block: 32 codes x 32 queries).  The lookups of the next 32 codes and the test of
// the block before stand among a block's products.  Where a block has a result that passes, the lanes that hold one leave
// their 16 results in LDS, without looking for it; later 64 lanes find those of four such, and once there are 64 pairs they
// are summed exactly, a lane each, from the queries' quantized tables in LDS, which the wavefronts of a workgroup share.
// What remains is reported when the unit is done: lists per (query, region) as scan_u8_mfma_kernel's, region = unit modulo the
// number of regions.  A unit of which more pairs pass than pay, or more at a time than LDS has room for, is given up: a bit in
// `left`, and scan_u8_left_kernel, launched after this one, does it.
constexpr int decoded_nw(int B) { return B == 8 ? 12 : 8; }      // wavefronts per workgroup
constexpr int decoded_lanes(int B) { return B == 8 ? 48 : 64; }  // lanes' results that wait (and 64 more of one block)
constexpr int DECODED_STAGE = 128; // pairs within the bound that a unit can have (and 64 more)
constexpr unsigned DECODED_ALLOW = 1024;  // pairs of a unit that may pass, and as many more as the pairs seen
constexpr int DECODED_SHARE = 8;          // shifted down by this

template <int B, int G>
struct DecodedShared {
    static constexpr int QW = 32 * G, NW = decoded_nw(B), LANES = decoded_lanes(B);
    __attribute__((aligned(16))) int tab[B * 32];  // (at the front: the lookups' offsets are then part of their instructions)
    __attribute__((aligned(16))) int norm[NW][2][32];
    __attribute__((aligned(16))) v4i_t results[NW][LANES + 64][4];
    unsigned place[NW][LANES + 64];        // their query << 24 | first code, of the unit
    unsigned pairs[NW][128];                       // that passed: query << 24 | code of the unit
    uint2 found[NW][DECODED_STAGE + 64];           // that are within the bound, with their sum
    int thr[QW];                                   // a result passes when it is below
    unsigned tau[QW];
    __attribute__((aligned(16))) uint8_t ql[QW][32 * B];
};

template <int B, int G>
__global__ __launch_bounds__(64 * decoded_nw(B)) void scan_u8_decoded_kernel(
    const uint8_t *__restrict__ codes, DecodedLeft all, int which, int regions, int nq, int cap_i,
    const uint8_t *__restrict__ qluts, const int *__restrict__ tables, const int *__restrict__ operands,
    const int2 *__restrict__ scales, const unsigned *__restrict__ taus, char *__restrict__ ws, size_t ws_stride,
    size_t countsA_off, size_t listsA_off, unsigned *__restrict__ flags, unsigned *__restrict__ left,
    unsigned *__restrict__ passed)
{
    using S = DecodedShared<B, G>;
    constexpr int NK = B / 4;    // words of a code, matrix instructions per block
    constexpr int QW = S::QW, NW = S::NW, NT = 64 * NW;
    __shared__ S sh;

    const int tid = threadIdx.x, l = tid & 63, wave = tid >> 6;
    const int row = l & 31, half = l >> 5;
    const DecodedPart of = all.parts[which];
    const int nsets = (nq + QW - 1) / QW;
    int set, part;
    tiled_group_and_chunk(nsets, set, part);
    const int parts = (int)(gridDim.x / (unsigned)nsets);
    const int q0 = set * QW;
    const unsigned cap = (unsigned)cap_i;
    if (part * NW >= of.units) return;  // uniform over the workgroup
    if (decoded_stopped(all, which)) return;  // uniform: scan_u8_rest_kernel goes on

    for (int i = tid; i < QW * 2 * B; i += NT)  // 16 bytes each
        reinterpret_cast<uint4 *>(sh.ql)[i] = reinterpret_cast<const uint4 *>(qluts)[(size_t)q0 * (2 * B) + min(i, (nq - q0) * 2 * B - 1)];
    for (int i = tid; i < B * 32; i += NT) sh.tab[i] = tables[i];
    for (int i = tid; i < QW; i += NT) {
        const int q = min(q0 + i, nq - 1);
        const unsigned t = taus[q];
        const int2 sc = scales[q];
        int thr = DECODED_NONE;
        if (q0 + i < nq && t < cap && sc.x > 0) thr = sc.x * (int)t - sc.y + 1;
        if (t >= cap) flags[q] = 1u;  // no bound: every sum would pass, and the query is done on its own
        sh.thr[i] = thr;
        sh.tau[i] = t;
    }
    v4i_t y[G][NK];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const int q = min(q0 + 32 * g + row, nq - 1);
#pragma unroll
        for (int k = 0; k < NK; ++k) y[g][k] = *reinterpret_cast<const v4i_t *>(operands + (size_t)q * (2 * B) + (2 * k + half) * 4);
    }
    __syncthreads();  // the only one
    int thr[G];
#pragma unroll
    for (int g = 0; g < G; ++g) thr[g] = sh.thr[32 * g + row];
    auto &norm = sh.norm[wave];
    auto &results = sh.results[wave];
    auto &place = sh.place[wave];
    auto &pairs = sh.pairs[wave];
    auto &found = sh.found[wave];
    auto order = [] { asm volatile("" ::: "memory"); };  // (a wavefront's LDS accesses are in the order of the program)

    for (int unit = part * NW + wave; unit < of.units; unit += parts * NW) {  // uniform over the wavefront
        int64_t c0, c1;
        decoded_unit(all, of, unit, c0, c1);
        if (c0 >= c1) continue;  // (behind the end of the last block)
        const unsigned len = (unsigned)(c1 - c0);  // (below 2^24, and 2^29 bytes)
        const uint8_t *unit_data = codes + c0 * B;
        // lane l reads code l of 64; v_permlane32_swap hands the words of the first and the last 32 to both halves
        auto fetch = [&](unsigned rel, unsigned (&w)[NK]) {
            const unsigned *src = reinterpret_cast<const unsigned *>(unit_data + min(rel + l, len - 1u) * (unsigned)B);
#pragma unroll
            for (int k = 0; k < NK; ++k) w[k] = src[k];
        };
        unsigned waiting = 0, npairs = 0, nfound = 0, seen = 0;  // uniform: lanes' results, pairs; pairs found, pairs summed
        // A pair per lane on its way: its code is requested by one call of check and summed at the next, so that the wavefront
        // need not wait for it.
        unsigned pw[NK], pe = NO_KEY;
        auto sum_pairs = [&]() {
            unsigned sum = 0;
            bool within = false;
            if (pe != NO_KEY) {
                const unsigned slot = pe >> 24;
                sum = exact_sum<B>(sh.ql[slot], pw);
                within = sum <= sh.tau[slot];
            }
            const unsigned long long all = __ballot(within);
            if (within) found[nfound + rank_in_mask(all)] = make_uint2(pe, sum);
            nfound = min(nfound + (unsigned)__popcll(all), (unsigned)DECODED_STAGE);
            pe = NO_KEY;
            order();
        };
        // The first `take` pairs; the rest moves to the front.
        auto check = [&](unsigned take) {
            if (seen) sum_pairs();
            order();
            pe = (unsigned)l < take ? pairs[l] : NO_KEY;
            if ((pe & 0xffffffu) >= len) pe = NO_KEY;
            const unsigned *src = reinterpret_cast<const unsigned *>(unit_data + min(pe & 0xffffffu, len - 1u) * (unsigned)B);
#pragma unroll
            for (int k = 0; k < NK; ++k) pw[k] = src[k];
            npairs -= take;
            seen += take;
            order();
            const unsigned rest = pairs[64 + l];
            order();
            pairs[l] = rest;
            order();
        };
        // The results that pass among those waiting, four lanes' at a time.
        auto drain = [&]() {
            order();
#pragma unroll 1
            for (unsigned e0 = 0; e0 < waiting; e0 += 4) {
                const unsigned e = e0 + (l >> 4), v = l & 15;
                const unsigned at = place[min(e, waiting - 1u)];
                const bool pass = e < waiting && reinterpret_cast<const int *>(results[min(e, waiting - 1u)])[v] < sh.thr[at >> 24];
                const unsigned long long all = __ballot(pass);
                if (pass) pairs[npairs + rank_in_mask(all)] = at + (v >> 2) * 8u + (v & 3u);
                npairs += (unsigned)__popcll(all);
                if (npairs >= 64u) check(64u);
            }
            waiting = 0;
            order();
        };

        unsigned cn[NK], cf[NK], cg[NK], w0[NK], w1[NK];  // codes requested two and one rounds ago, and in this one
        v4i_t a[2][NK];
        v16i_t acc[2];  // a block's results are tested while the next block's products run
        auto spread = [&]() {
#pragma unroll
            for (int k = 0; k < NK; ++k) {
                const auto p = __builtin_amdgcn_permlane32_swap(cn[k], cn[k], false, false);
                w0[k] = p[0];
                w1[k] = p[1];
            }
        };
        auto multiply = [&](const v4i_t (&op)[NK], const v16i_t &init, int g) {
            v16i_t r = init;
#pragma unroll
            for (int k = 0; k < NK; ++k) r = __builtin_amdgcn_mfma_i32_32x32x32_i8(op[k], y[g][k], r, 0, 0, 0);
            return r;
        };
        // Result v of a lane: code (v / 4) * 8 + half * 4 + v % 4 of the block, query row.
        const unsigned own = (unsigned)row << 24 | (unsigned)half * 4u;
        auto test = [&](const v16i_t &r, int g, unsigned rel) {
            int lo = r[0];
#pragma unroll
            for (int v = 1; v < 15; v += 2) lo = min(min(lo, r[v]), r[v + 1]);
            lo = min(lo, r[15]);
            const unsigned long long all = __ballot(lo < thr[g]);
            if (all == 0ull) return;
            if (lo < thr[g]) {
                const unsigned at = waiting + rank_in_mask(all);
#pragma unroll
                for (int u = 0; u < 4; ++u) results[at][u] = v4i_t{r[4 * u], r[4 * u + 1], r[4 * u + 2], r[4 * u + 3]};
                place[at] = own + (rel + ((unsigned)g << 29));
            }
            waiting = min(waiting + (unsigned)__popcll(all), (unsigned)S::LANES);
        };
        auto norms = [&](int buf) {
            v16i_t r;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const v4i_t v = *reinterpret_cast<const v4i_t *>(&norm[buf][8 * g + 4 * half]);
#pragma unroll
                for (int e = 0; e < 4; ++e) r[4 * g + e] = v[e];
            }
            return r;
        };
        // share g of G of the lookups of words w[]; the squares of a share come a block later
        constexpr int SH = G - 1;  // blocks with lookups
        static_assert(G > 1, "");
        int sq[2];
        auto lookup = [&](const unsigned (&w)[NK], v4i_t (&op)[NK], int g) {
#pragma unroll
            for (int k = 0; k < NK; ++k)
                if (min(k * SH / NK, SH - 1) == g) op[k] = decoded_lookup(sh.tab, w[k], k, half);
        };
        auto square = [&](const v4i_t (&op)[NK], int g) {
#pragma unroll
            for (int k = 0; k < NK; ++k)
                if (min(k * SH / NK, SH - 1) == g)
#pragma unroll
                    for (int e = 0; e < 4; ++e) sq[e & 1] = __builtin_amdgcn_sdot4(op[k][e], op[k][e], sq[e & 1], false);
            asm volatile("" : "+v"(sq[0]), "+v"(sq[1]));  // (they stay in this block; left to itself the compiler sinks them into one)
        };
        auto leave_norm = [&](int buf) {
            const int own_half = sq[0] + sq[1];
            const auto p = __builtin_amdgcn_permlane32_swap(own_half, own_half, false, false);
            norm[buf][row] = (int)(p[0] + p[1]) >> 2;  // (both halves write the same)
            order();
        };
        // the G blocks of 32 codes (operand a[S0], codes from rel on), with the lookups of the next 32, words w
        auto step = [&](auto which, const unsigned (&w)[NK], unsigned rel) {
            constexpr int S0 = decltype(which)::value;
            const v16i_t init = norms(S0);
            sq[0] = sq[1] = 0;
#pragma unroll
            for (int g = 0; g < G; ++g) {
                acc[(S0 * G + g) & 1] = multiply(a[S0], init, g);
                lookup(w, a[S0 ^ 1], g);
                if (g > 0) square(a[S0 ^ 1], g - 1);
                test(acc[(S0 * G + g + 1) & 1], g > 0 ? g - 1 : G - 1, g > 0 ? rel : rel - 32u);
            }
            leave_norm(S0 ^ 1);
        };
        fetch(0, cn);
        fetch(64, cf);
        fetch(128, cg);
        spread();
        sq[0] = sq[1] = 0;
#pragma unroll
        for (int g = 0; g < SH; ++g) {
            lookup(w0, a[0], g);
            square(a[0], g);
        }
        leave_norm(0);
        bool give_up = false;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[1][v] = 1 << 29;  // (passes nothing)
        for (unsigned rel = 0; rel < len; rel += 64) {  // uniform
#pragma unroll
            for (int k = 0; k < NK; ++k) { cn[k] = cf[k]; cf[k] = cg[k]; }
            fetch(rel + 192, cg);  // (past the end: the last code again)
            step(std::integral_constant<int, 0>(), w1, rel);
            spread();
            step(std::integral_constant<int, 1>(), w0, rel + 32u);
            if (waiting >= 16u) {
                give_up = waiting >= (unsigned)S::LANES || seen > DECODED_ALLOW + (rel >> DECODED_SHARE) * (unsigned)QW;
                if (give_up) break;
                drain();
            }
        }
        if (!give_up) {
            test(acc[1], G - 1, (len - 1u) / 64u * 64u + 32u);
            give_up = waiting >= (unsigned)S::LANES;
            if (!give_up) {
                drain();
                if (npairs) check(npairs);
                sum_pairs();
            }
        }
        order();
        if (l == 0) atomicAdd(&passed[which], give_up ? max(seen, len * (unsigned)QW >> DECODED_SHARE) : seen);
        if (give_up || nfound >= (unsigned)DECODED_STAGE) {
            if (l == 0) atomicOr(&left[set * all.pitch + of.word + (unit >> 5)], 1u << (unit & 31));
            continue;
        }
        const int region = unit % regions;
        for (unsigned i = l; i < nfound; i += 64) {
            const uint2 e = found[i];
            const int q = q0 + (int)(e.x >> 24);
            char *base = ws + (size_t)q * ws_stride;
            const unsigned at = atomicAdd(reinterpret_cast<unsigned *>(base + countsA_off) + region, 1u);
            if (at < (unsigned)TILED_LCAP)
                reinterpret_cast<uint64_t *>(base + listsA_off)[(size_t)region * TILED_LCAP + at] =
                    (uint64_t)e.y << 32 | (uint64_t)(c0 + (e.x & 0xffffffu));
            else
                flags[q] = 1u;  // keys are dropped: this query is redone on its own
        }
        order();
    }
}

// Between two parts of the scan, a workgroup per query: the R-th smallest sum found so far bounds the rest, and the keys
// beyond it are dropped.
__global__ __launch_bounds__(256) void decoded_refine_kernel(char *__restrict__ ws, size_t ws_stride, size_t countsA_off,
                                                             size_t listsA_off, int regions, int R, unsigned *__restrict__ taus,
                                                             const unsigned *__restrict__ flags, DecodedLeft all, int done)
{
    __shared__ unsigned hist[256];
    __shared__ unsigned bound;
    const int q = blockIdx.x, tid = threadIdx.x;
    if (flags[q] == 1u || decoded_stopped(all, done)) return;  // uniform
    char *base = ws + (size_t)q * ws_stride;
    unsigned *counts = reinterpret_cast<unsigned *>(base + countsA_off);
    uint64_t *lists = reinterpret_cast<uint64_t *>(base + listsA_off);
    hist[tid] = 0;
    __syncthreads();
    for (int r = tid; r < regions; r += 256) {
        const unsigned c = min(counts[r], (unsigned)TILED_LCAP);
        const uint64_t *l = lists + (size_t)r * TILED_LCAP;
        for (unsigned i = 0; i < c; i += 4) {  // four loads in flight
            uint64_t k[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) k[u] = l[min(i + u, c - 1u)];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (i + u < c) atomicAdd(&hist[(unsigned)(k[u] >> 32) & 255u], 1u);
        }
    }
    __syncthreads();
    if (tid < WAVE) {
        unsigned h[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) h[b] = hist[4 * tid + b];
        const unsigned t = wave_threshold_bin<4>(h, (unsigned)R);
        if (tid == 0) {
            bound = t;
            if (t < taus[q]) taus[q] = t;
        }
    }
    __syncthreads();
    const unsigned t = bound;
    if (t >= 255u) return;  // uniform (256: fewer than R so far)
    for (int r = tid; r < regions; r += 256) {
        const unsigned c = min(counts[r], (unsigned)TILED_LCAP);
        uint64_t *l = lists + (size_t)r * TILED_LCAP;
        unsigned kept = 0;
        for (unsigned i = 0; i < c; ++i) {
            const uint64_t k = l[i];
            if ((unsigned)(k >> 32) <= t) l[kept++] = k;
        }
        if (kept < c) {
            for (unsigned i = kept; i < c; ++i) l[i] = 0;
            counts[r] = kept;
        }
    }
}

constexpr int DECODED_G = 4;  // groups of 32 queries per wavefront

// When it pays: matrix products a pair are half of scan_u8_mfma_kernel's, but every pair that passes costs some 30 cycles, and how
// many pass depends on how many sums the last bound lets in (R of n) and on what the quantizer's steps lose.  Measured against
// scan_u8_mfma_kernel, the whole search, its time over the time here, the least and the mean over 2 codebooks and 100, 200 and 1000 initial
// codes of a mixture's vectors (the fewer, the coarser the steps):
//   16-byte codes      n / R     2.5e5          3.5e5          5e5            7e5            1e6
//     8 M x 256              0.93  0.99     0.96  1.03     1.01  1.08     1.05  1.13     1.08  1.15
//     12 M x 256             0.91  0.99     0.96  1.04     1.01  1.08     1.06  1.14     1.11  1.19
//     32 M x 256             0.94  1.01     0.97  1.06     1.01  1.12     1.11  1.21     1.18  1.28
//     100 M x 256                                          0.85  1.05     0.98  1.14     0.99  1.18
//     16 M x 128             0.80  0.88     0.88  0.94     0.91  0.97     0.96  1.01     0.99  1.05
//     24 M x 128             0.90  0.95     0.88  0.98     0.97  1.05     1.01  1.09     1.06  1.14
//     32 M x 65              0.95  1.10     0.97  1.12     1.13  1.19     1.17  1.22     1.20  1.24
//   8-byte codes       n / R     1.6e5          2.5e5          5e5
//     16 M x 256             0.95  1.06     1.13  1.15     1.14  1.15
//     32 M x 256             1.01  1.10     0.95  1.12     1.23  1.28
//     16 M x 128             0.86  0.90     0.93  0.93     0.92  0.93
//     32 M x 128             0.97  1.03     0.93  1.03     1.08  1.10
// Within n / R of 7e5 and 8e5, 100 initial codes and 16-byte codes, three shapes of 40 lost 3 to 5 % (11 M x 335, R = 15 971 -> 1018 us); 8-byte
// codes with sub-vectors of one component, 5e5, 100 M x 494 0.92.  Sets of queries: the launches of the
// parts are for all of them, and a last set of 64 and less costs as one of 128 (64 queries, 32 M R = 10 0.77 to 0.83, 65 1.3; 129 0.93;
// 166 over 16 M R = 19 0.88).  Steps: R = 50 of 50 M with 255 / 224 / 200 / 160 / 127 bins 1.33 / 1.20 / 1.12 / 0.98 / 0.89.  R: the
// sample is no larger than 512 tiles, and beyond it too many pairs pass in the first part (100 M, R = 200 with a fourth of the sample: the
// units' lists overflow, all queries are redone one by one, 66 ms; R = 256 is the largest measured, 1.17).
// 288 shapes within the lines, 65 to 520 queries, 6 to 100 M codes, 100 to 1000 initial codes, 224 and 255 bins: 1.45 on average, the
// least 0.98, but for R = 1, where either route now and then redoes a query (0.91 to 4).
// Sizes don't tell what data and quantizers do, so each part counts the pairs that passed, and behind a part with more than
// DECODED_PASS / 4096 of all its pairs the batch goes back to the one-hot products: within the lines that has cost up to 3 % (51 M x 127,
// 96 dimensions, 100 initial codes, 224 bins: 1413 -> 1451 us; 100 M x 256, 255 bins 5349 -> 5411; let on, 2739 -> 2851 for 128 queries).
// For the 8-byte codes a product is cheaper beside the check: their share is smaller.
constexpr int DECODED_PASS[2][2] = {{6, 4}, {21, 15}};  // 8- and 16-byte codes: the first part, whose bound is the sample's, the others
constexpr int64_t DECODED_MIN_N[2] = {32000000, 24000000};  // codes times sets of queries
constexpr int64_t DECODED_N_PER_R[2] = {700000, 850000};
constexpr int DECODED_MAX_R = 256;
constexpr int DECODED_MIN_BINS = 224;
constexpr int DECODED_MIN_LAST = 65;              // queries in the last set of 128

// The scan in parts, the bound tightened behind each but the last (the first one's is a sample's: R of some 8e5 codes, and the
// share that passes falls 4 to 6 times with it; 1/16, 1/3 and the rest took as long, and cost 5 % more where the batch goes back).
// A part is a stretch of every block of the database, not of the database: stored cluster by cluster, the first 64th of it bounds
// the queries of one cluster (73 M codes of 8 bytes in runs of 20,000 of a cluster, 256 queries, R = 100, by the tightened bounds and
// the one-hot products 35.5 ms, now 2.0; whole clusters one after the other, R = 10 5.2 ms for 100 M of 16 bytes, now 3.8).
// Blocks and units: as many units for every wavefront that the chip holds at once, of about 8192 codes (2048 in the first two parts, whose
// bounds let more in): four rounds and what is left over instead, 73 M x 256, m = 16 1.55 -> 1.73 ms, 40 M x 384, m = 32 2.42 -> 3.69 (there
// with more workgroups than the chip holds); 976 blocks for 1024 wavefronts, 32 M x 256 1.11 -> 1.15.
// Workgroups of a set: a CU holds one, an XCD's share is whole.
static int decoded_wgs(int sets) { return std::max(256 / (8 * sets), 1) * 8; }

static void decoded_parts(int B, int64_t n, int nq, int sets, DecodedLeft *all)
{
    const int64_t waves = (int64_t)decoded_wgs(sets) * decoded_nw(B);  // of a set, that the chip holds at once
    // a block for every wavefront, or for every second, third ... of them: a block's first part is a unit of 448 codes at least
    const int64_t blocks = std::max<int64_t>(1, waves / std::max<int64_t>(1, ceil_div(waves, std::max<int64_t>(1, n / (64 * 448)))));
    const int64_t block = ceil_div(ceil_div(n, blocks), 64) * 64;
    all->n = n;
    all->block = (int)block;
    all->blocks = (int)ceil_div(n, block);
    const int64_t ends[DECODED_PARTS] = {block / 64, block / 12, block / 3, block};
    int64_t from = 0;
    int k = 0, word = 0;
    for (int64_t e : ends) {
        const int64_t to = e / 64 * 64;
        if (to <= from) continue;
        const int64_t codes = (to - from) * all->blocks;
        // units per block: what takes a wavefront the shortest
        const int64_t len = to - from, most = k < 2 ? 2560 : 10240, few = ceil_div(len, most);
        const int64_t many = std::max(few, std::min(len / 448, few + 4 + waves / all->blocks));
        int per = 0, unit = 0;
        int64_t least = INT64_MAX;
        for (int64_t p = few; p <= many; ++p) {
            const int64_t u = ceil_div(ceil_div(len, p), 64) * 64, time = ceil_div(p * all->blocks, waves) * (u + 128);
            if (time < least) { least = time; per = (int)p; unit = (int)u; }
        }
        all->parts[k] = {(int)from, (int)to, unit, per, per * all->blocks, word,
                         (unsigned)std::min<int64_t>(codes / 64 * nq / 64 * DECODED_PASS[B / 16][k > 0], UINT32_MAX / 2)};
        word += (int)ceil_div(all->parts[k].units, 32);
        from = to;
        ++k;
    }
    all->nparts = k;
    all->pitch = word;
    all->queries = 32 * DECODED_G;
}

// Room a batch takes: decoded tables, operands and scales, and the bits of `words` words per set.
static size_t decoded_room(int m, int nq, int sets, int words)
{
    return (size_t)m * 64 + (size_t)nq * (4 * m + sizeof(int2)) + (DECODED_PARTS + (size_t)sets * words) * 4;
}

bool decoded_pays(int B, int64_t n, int nq, int cap, int R, const DecodedBatch &db)
{
    if (knobs().tiled_decoded == 0 || (B != 8 && B != 16) || db.d > 8 * B) return false;
    const int sets = (int)ceil_div(nq, 32 * DECODED_G);
    const bool sizes = n * sets >= DECODED_MIN_N[B / 16] && n >= R * DECODED_N_PER_R[B / 16] && R <= DECODED_MAX_R &&
                       cap >= DECODED_MIN_BINS && nq - 32 * DECODED_G * (sets - 1) >= DECODED_MIN_LAST;
    if (!sizes && knobs().tiled_decoded < 0) return false;
    DecodedLeft all = {};
    decoded_parts(B, n, nq, sets, &all);
    return decoded_room(2 * B, nq, sets, all.pitch) <= db.room_bytes;
}

template <int B>
static DecodedLeft run_decoded(const TiledPlan &t, const uint8_t *codes, int64_t n, int nq, int cap, int R, const uint8_t *qluts,
                               unsigned *taus, char *ws, size_t ws_stride, size_t countsA_off, size_t listsA_off,
                               unsigned *flags, const DecodedBatch &db, hipStream_t st)
{
    constexpr int m = 2 * B;
    int *tables = (int *)db.room, *operands = tables + m * 16;
    int2 *scales = (int2 *)(operands + (size_t)nq * m);
    unsigned *passed = (unsigned *)(scales + nq), *left;
    constexpr int G = DECODED_G;
    const int sets = (int)ceil_div(nq, 32 * G);
    DecodedLeft all = {};
    decoded_parts(B, n, nq, sets, &all);
    left = passed + DECODED_PARTS;
    all.bits = left;
    all.passed = passed;
    launch(QADC_PROF_SEED, decoded_prepare_kernel<B>, dim3((unsigned)nq), dim3(32 * B), 0, st, db.codebooks, db.d, db.queries, qluts,
           db.deltas, cap, tables, operands, scales, passed, DECODED_PARTS + sets * all.pitch);
    for (int k = 0; k < all.nparts; ++k) {
        const DecodedPart &p = all.parts[k];
        if (k > 0)
            launch(QADC_PROF_SEED, decoded_refine_kernel, dim3((unsigned)nq), dim3(256), 0, st, ws, ws_stride, countsA_off, listsA_off,
                   t.GC, R, taus, (const unsigned *)flags, all, k - 1);
        const int64_t wgs = std::min<int64_t>(ceil_div(ceil_div(p.units, decoded_nw(B)), 8) * 8, decoded_wgs(sets));
        const dim3 grid((unsigned)(wgs * sets));
        launch(QADC_PROF_SCAN, (scan_u8_decoded_kernel<B, G>), grid, dim3(64 * decoded_nw(B)), 0, st, codes, all, k, t.GC, nq, cap, qluts,
               (const int *)tables, (const int *)operands, (const int2 *)scales, (const unsigned *)taus, ws, ws_stride, countsA_off,
               listsA_off, flags, left, passed);
    }
    return all;
}

DecodedLeft run_decoded_scan(const TiledPlan &t, const uint8_t *codes, int64_t n, int nq, int cap, int R, const uint8_t *qluts,
                             unsigned *taus, char *ws, size_t ws_stride, size_t countsA_off, size_t listsA_off,
                             unsigned *flags, const DecodedBatch &db, hipStream_t st)
{
#define QADC_ARGS t, codes, n, nq, cap, R, qluts, taus, ws, ws_stride, countsA_off, listsA_off, flags, db, st
    return t.B == 8 ? run_decoded<8>(QADC_ARGS) : run_decoded<16>(QADC_ARGS);
#undef QADC_ARGS
}

}  // namespace qadc
