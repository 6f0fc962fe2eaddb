// Pieces shared by the scan kernels of the Quick ADC library (gfx950): workspace layout,
// tile loads, candidate-list compaction, the cross-workgroup merge kernel.
#pragma once

#include <stdlib.h>

#include "qadc_select.h"
#include "qadc_profile.h"

namespace qadc {

constexpr int SCAN_VEC = 2;               // 16-byte loads per thread and tile
constexpr int SCAN_SLACK = QADC_MAX_R;    // candidate slots beyond one tile
constexpr int GH_REP = 2;                 // replicas of the grid-wide histogram
constexpr unsigned NO_KEY = 0xffffffffu;
constexpr unsigned IVFS_NONE = 0xffffffffu;  // a query of the shared-list scan without a bound

// Per-query control block in the workspace, followed by counts[G] (keys reported by each
// workgroup) and lists[G][R] (the keys).  Block and counts must be all zero when the scan
// kernel starts; the merge kernel leaves every word the call wrote zeroed again.
struct alignas(256) ScanHeader {
    unsigned ghist[GH_REP][256];  // sums of the best codes of every seed tile
    uint8_t ptab[32 * 256];       // the query's pair tables, left by the seed kernel for the scan
};

// Geometry of a scan.  B = bytes per code for 4-bit components (two per byte; also for 8-bit
// components, one per byte); B = SIXBIT + m for codes of m 6-bit components (3m/4 bytes, stored
// back to back, least significant bit first), whose thread takes 48 contiguous bytes per tile.
constexpr int SIXBIT = 1000;
template <int B, int NT>
struct ScanCfg {
    static constexpr bool SIX = B >= SIXBIT;
    static constexpr int M6 = SIX ? B - SIXBIT : 0;               // 6-bit components per code
    static constexpr int BYTES = SIX ? 3 * M6 / 4 : B;            // bytes per code
    static constexpr int NVEC = SIX ? 3 : SCAN_VEC;               // 16-byte loads per thread and tile
    static constexpr int CPV = (!SIX && B <= 16) ? 16 / B : 1;    // codes per 16-byte load (4-bit)
    static constexpr int CPT = SIX ? 48 / BYTES : ((B <= 16) ? SCAN_VEC * CPV : 1);  // codes per thread and tile
    static constexpr int TILE = NT * CPT;
    static constexpr int CAP = TILE + SCAN_SLACK;
    static constexpr int TAB_BYTES = SIX ? M6 * 64 : B * 256;     // lookup tables of a query in LDS
};

__device__ __forceinline__ unsigned byte_of(const uint4 &v, int k)
{
    const unsigned w = (k < 4) ? v.x : (k < 8) ? v.y : (k < 12) ? v.z : v.w;
    return (w >> (8 * (k & 3))) & 0xffu;
}

// Keys with sum <= tau are exactly the keys below this limit.
__device__ __forceinline__ unsigned limit_of_bin(unsigned tau)
{
    return tau >= 255u ? NO_KEY : ((tau + 1u) << 24);
}

// Called by one whole wave; h[b] is the count of bin NB*lane+b.  Returns, in every lane,
// the smallest bin whose inclusive running count reaches `need`, or 64*NB when none does.
template <int NB>
__device__ __forceinline__ unsigned wave_threshold_bin(const unsigned (&h)[NB], unsigned need,
                                                       unsigned *total = nullptr)
{
    const int l = lane_id();
    unsigned tot = 0;
#pragma unroll
    for (int b = 0; b < NB; ++b) tot += h[b];
    const unsigned inc = wave_running_sum(tot);
    if (total) *total = lane_value(inc, WAVE - 1);
    const unsigned long long m = __ballot(inc >= need);
    if (m == 0) return (unsigned)(WAVE * NB);
    const int first = __ffsll((long long)m) - 1;
    unsigned run = inc - tot, bin = (unsigned)(NB * l + NB - 1);
    bool found = false;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        run += h[b];
        if (!found && run >= need) { bin = (unsigned)(NB * l + b); found = true; }
    }
    return lane_value(bin, first);
}

// Cuts keys[0..cnt) back to its `keep` smallest keys and returns the largest key kept.  A list
// of at most `keep` keys is left as it is (the value returned then bounds nothing).  K = key
// type, NBYTES = key bytes that can be non-zero.  Called by every thread of the workgroup with
// the same cnt and keep; `ccnt` is an LDS counter of the workgroup.  The caller's list then
// holds min(cnt, keep) keys.
template <typename K, int NBYTES, int NT, int CAP>
__device__ K compact_candidates(K *keys, unsigned cnt, unsigned keep, SelectScratch *sel,
                                unsigned *ccnt)
{
    if (cnt <= keep) return ~(K)0 - 1;  // uniform
    const K kth = block_radix_select<K, NBYTES>(keys, cnt, keep, sel);
    constexpr int PER = (CAP + NT - 1) / NT;
    K mine[PER];
#pragma unroll
    for (int t = 0; t < PER; ++t) {
        unsigned i = threadIdx.x + t * NT;
        mine[t] = (i < cnt) ? keys[i] : ~(K)0;
    }
    if (threadIdx.x == 0) *ccnt = 0;
    __syncthreads();
#pragma unroll
    for (int t = 0; t < PER; ++t) {
        unsigned i = threadIdx.x + t * NT;
        bool ok = (i < cnt) && (mine[t] <= kth);
        unsigned slot = wave_append_slot(ok, ccnt);
        if (ok) keys[slot] = mine[t];
    }
    __syncthreads();
    return kth;
}

// 16-byte streaming load: the codes are read once per query, so they are fetched with the
// non-temporal hint and do not displace the tables and candidate lists from the caches.
typedef unsigned v4u __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 stream_load16(const uint8_t *p)
{
    const v4u v = __builtin_nontemporal_load(reinterpret_cast<const v4u *>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}

// 12-byte streaming load (the address is a multiple of four).
typedef unsigned v3u __attribute__((ext_vector_type(3)));
typedef v3u v3u_a4 __attribute__((aligned(4)));
__device__ __forceinline__ v3u stream_load12(const uint8_t *p)
{
    return __builtin_nontemporal_load(reinterpret_cast<const v3u_a4 *>(p));
}

// How a wavefront shares out its 64 * 48 bytes of 6-bit codes: in groups of whole codes of 12 or
// 24 bytes, group g of lane l being group 64 g + l of the wavefront's bytes, so that one load
// instruction reads consecutive groups.  The thread keeps its groups one after the other: code c of
// the thread starts at byte c * BYTES of its 48 bytes and is code
// (64 (c / CPG) + l) * CPG + c % CPG of the wavefront.
template <int BYTES>
struct SixbitLayout {
    static constexpr int UPG = BYTES > 12 ? BYTES / 12 : 1;   // 12-byte loads per group
    static constexpr int CPG = BYTES > 12 ? 1 : 12 / BYTES;   // codes per group
    static constexpr int GROUPS = 4 / UPG;                    // groups per thread and tile
    static_assert(BYTES == 6 || BYTES == 12 || BYTES == 24, "6-bit codes of 8, 16 or 32 components");
    // index of code c of thread `tid` inside the tile
    static __device__ __forceinline__ unsigned slot(int tid, int c)
    {
        constexpr int CPT = 48 / BYTES;
        return (unsigned)((tid & ~(WAVE - 1)) * CPT + ((c / CPG) * WAVE + (tid & (WAVE - 1))) * CPG + c % CPG);
    }
};

// The two 16-byte loads of one thread for the tile starting at code t0 (6-bit components: its
// four groups, as three vectors).  FULL: the whole
// tile lies inside the database (t0 + TILE <= c1), no bounds to check.
template <int B, int NT, bool FULL = false>
__device__ __forceinline__ void tile_load(const uint8_t *__restrict__ codes, int64_t t0, int64_t c1,
                                          uint4 (&w)[ScanCfg<B, NT>::NVEC], int (&nc)[2])
{
    const int tid = threadIdx.x;
    if constexpr (ScanCfg<B, NT>::SIX) {
        // 6-bit components: four groups of 12 or 24 bytes per thread (sixbit_layout); nc[0] = bit c
        // set when code c of the thread lies inside the database
        using C = ScanCfg<B, NT>;
        using L = SixbitLayout<C::BYTES>;
        const int64_t wave0 = t0 + (int64_t)(tid & ~(WAVE - 1)) * C::CPT;  // first code of the wavefront
        const int lane = tid & (WAVE - 1);
        unsigned d[12];
        nc[0] = 0;
        nc[1] = 0;
#pragma unroll
        for (int g = 0; g < L::GROUPS; ++g) {
            const int64_t first = wave0 + (int64_t)(g * WAVE + lane) * L::CPG;  // first code of the group
            const uint8_t *p = codes + first * C::BYTES;
            if (FULL || first + L::CPG <= c1) {
#pragma unroll
                for (int u = 0; u < L::UPG; ++u) {
                    const v3u v = stream_load12(p + 12 * u);
                    d[(g * L::UPG + u) * 3] = v.x;
                    d[(g * L::UPG + u) * 3 + 1] = v.y;
                    d[(g * L::UPG + u) * 3 + 2] = v.z;
                }
                nc[0] |= ((1 << L::CPG) - 1) << (g * L::CPG);
            } else {  // ragged end of the database: byte loads, no read past the end
                const int have = first < c1 ? (int)(c1 - first) : 0;
                unsigned tmp[3 * L::UPG];
#pragma unroll
                for (int k = 0; k < 3 * L::UPG; ++k) tmp[k] = 0;
                for (int k = 0; k < have * C::BYTES; ++k) tmp[k >> 2] |= (unsigned)p[k] << (8 * (k & 3));
#pragma unroll
                for (int k = 0; k < 3 * L::UPG; ++k) d[g * L::UPG * 3 + k] = tmp[k];
                nc[0] |= ((1 << have) - 1) << (g * L::CPG);
            }
        }
#pragma unroll
        for (int v = 0; v < 3; ++v) w[v] = make_uint4(d[4 * v], d[4 * v + 1], d[4 * v + 2], d[4 * v + 3]);
    } else if constexpr (FULL) {
        if constexpr (B <= 16) {
            constexpr int CPV = 16 / B;
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                w[v] = stream_load16(codes + (t0 + ((int64_t)v * NT + tid) * CPV) * B);
                nc[v] = CPV;
            }
        } else {
            w[0] = stream_load16(codes + (t0 + tid) * B);
            w[1] = stream_load16(codes + (t0 + tid) * B + 16);
            nc[0] = 1;
            nc[1] = 0;
        }
    } else if constexpr (B <= 16) {
        constexpr int CPV = 16 / B;
#pragma unroll
        for (int v = 0; v < 2; ++v) {
            const int64_t base = t0 + ((int64_t)v * NT + tid) * CPV;
            w[v] = make_uint4(0, 0, 0, 0);
            nc[v] = 0;
            if (base + CPV <= c1) {
                w[v] = stream_load16(codes + base * B);
                nc[v] = CPV;
            } else if (base < c1) {  // ragged end of the database: byte loads, no read past the end
                nc[v] = (int)(c1 - base);
                unsigned tmp[4] = {0, 0, 0, 0};
                for (int k = 0; k < nc[v] * B; ++k)
                    tmp[k >> 2] |= (unsigned)codes[base * B + k] << (8 * (k & 3));
                w[v] = make_uint4(tmp[0], tmp[1], tmp[2], tmp[3]);
            }
        }
    } else {
        const int64_t i = t0 + tid;
        w[0] = w[1] = make_uint4(0, 0, 0, 0);
        nc[0] = nc[1] = 0;
        if (i < c1) {
            w[0] = stream_load16(codes + i * B);
            w[1] = stream_load16(codes + i * B + 16);
            nc[0] = 1;
        }
    }
}

// Sixteen entries of a pair table, min(cap, low[v] + high) for v = 0 .. 15: a thread makes a row of 16 bytes with 33
// vector instructions and writes it at once (an entry at a time, the LDS was busy for some 1000 cycles per 4096 entries).
__device__ __forceinline__ uint4 pair_row(const uint4 &low, unsigned high, unsigned cap)
{
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    const unsigned h = high | (high << 16), c = cap | (cap << 16);
    auto four = [&](unsigned w) {
        const unsigned even = (w & 0x00ff00ffu) + h, odd = ((w >> 8) & 0x00ff00ffu) + h;  // (at most 510 each: no carry)
        const u16x2 e = __builtin_elementwise_min(__builtin_bit_cast(u16x2, even), __builtin_bit_cast(u16x2, c));
        const u16x2 o = __builtin_elementwise_min(__builtin_bit_cast(u16x2, odd), __builtin_bit_cast(u16x2, c));
        return __builtin_bit_cast(unsigned, e) | (__builtin_bit_cast(unsigned, o) << 8);
    };
    return make_uint4(four(low.x), four(low.y), four(low.z), four(low.w));
}

// Pair tables ptab[jb][v] = min(cap, q[2jb][v & 15] + q[2jb + 1][v >> 4]) from a query's tables in LDS (both 16-byte
// aligned), by NT threads.
template <int B, int NT>
__device__ __forceinline__ void pair_rows_from_lds(const uint8_t *qlut_s, unsigned cap, uint8_t *ptab)
{
    for (int e = threadIdx.x; e < B * 16; e += NT) {
        const int jb = e >> 4;
        const uint4 low = *reinterpret_cast<const uint4 *>(qlut_s + 2 * jb * 16);
        reinterpret_cast<uint4 *>(ptab)[e] = pair_row(low, qlut_s[(2 * jb + 1) * 16 + (e & 15)], cap);
    }
}

// Order-preserving map float -> unsigned (any sign), and back.
__device__ __forceinline__ unsigned f2ord(float f)
{
    const unsigned b = __float_as_uint(f);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float ord2f(unsigned o)
{
    return __uint_as_float((o & 0x80000000u) ? (o & 0x7fffffffu) : ~o);
}


// ---------------------------------------------------------------- merge

constexpr int MERGE_NT = 1024;
constexpr int MERGE_CAP = 6144;   // keys staged in LDS
constexpr int MERGE_WG_PER_THREAD = 8;
constexpr int MERGE_FLAT_G = 256;        // regions and ...
constexpr int MERGE_FLAT_SLOTS = 32768;  // ... key slots up to which every slot is visited

// R best of the keys reported by the G workgroups of each query (64-bit keys
// dist << 32 | index, at most R per workgroup), ordered; then everything the call wrote
// in the workspace is cleared.  KBYTES = significant key bytes (5 for u8 distances).
// DistT = uint8_t: the distance is the key's bits 32..39; float: bits 32..63 (ordered image).
//
// Usual case (a few hundred to a few thousand keys in all): the keys are gathered in LDS; one
// histogram pass over the eight most significant bits in which they differ at all finds the
// bin of the R-th key; the keys up to that bin are ranked against each other by counting,
// which selects and orders in one step.  Massive ties fall back to the full radix select.
// Two report regions may exist per query: region B (G workgroups, up to R keys each) written
// by the single-query kernels, and region A (GA workgroups, up to pitchA keys each) written
// by the query-tiled kernel.  flags[q]: 0 = region A holds the result of query q; 1 = region A is
// incomplete and region B holds the result; 2 = the result is spread over both regions (the lists
// of an inverted index scanned partly by one kernel, partly by the other).  Without flags only
// region B exists.
// VISIT: regions that are few and well filled are gathered slot by slot (not for sparse ones).
template <typename DistT, int KBYTES, bool VISIT>
__global__ __launch_bounds__(MERGE_NT) void merge_topk_kernel(
    char *__restrict__ ws, size_t ws_stride, size_t counts_off, size_t lists_off, int G,
    unsigned need, int R, DistT pad_dist, uint32_t *__restrict__ out_idx,
    DistT *__restrict__ out_dist, size_t countsA_off, size_t listsA_off, int GA, int pitchA,
    unsigned *__restrict__ flags, const uint32_t *__restrict__ ids, int64_t n_ids)
{
    // need = min(R, number of codes scanned): at least that many keys were reported.
    // ids: the keys' low words are storage positions and out_idx gets ids[position] (inverted index).
    __shared__ uint64_t lkeys[MERGE_CAP];
    __shared__ uint64_t cand[MERGE_NT];
    __shared__ SelectScratch sc;
    __shared__ unsigned lcnt, ccnt;
    __shared__ unsigned long long all_or, all_and;
    __shared__ unsigned fcnt[MERGE_FLAT_G];

    const int tid = threadIdx.x;
    const int q = blockIdx.x;
    ScanHeader *hdr = reinterpret_cast<ScanHeader *>(ws + (size_t)q * ws_stride);
    unsigned *counts = reinterpret_cast<unsigned *>(ws + (size_t)q * ws_stride + counts_off);
    uint64_t *lists = reinterpret_cast<uint64_t *>(ws + (size_t)q * ws_stride + lists_off);
    int pitch = R;
    const unsigned flag = flags ? flags[q] : 1u;  // uniform
    const bool redone = flags && flag == 1u;
    const bool both = flag == 2u;
    unsigned *countsA = reinterpret_cast<unsigned *>(ws + (size_t)q * ws_stride + countsA_off);
    uint64_t *listsA = reinterpret_cast<uint64_t *>(ws + (size_t)q * ws_stride + listsA_off);
    if (flag == 0u) {                             // the tiled kernel's report is the result
        counts = reinterpret_cast<unsigned *>(ws + (size_t)q * ws_stride + countsA_off);
        lists = reinterpret_cast<uint64_t *>(ws + (size_t)q * ws_stride + listsA_off);
        G = GA;
        pitch = pitchA;
    }
    // Few, well-filled regions (inverted-index scans, short databases): every slot of every
    // region is visited, a slot per thread at a time, so that the loads are spread over the whole
    // workgroup instead of one thread walking each region.
    const bool flat = VISIT && G <= MERGE_FLAT_G && (size_t)G * pitch <= (size_t)MERGE_FLAT_SLOTS;  // uniform
    // every reported key, spread over the threads by workgroup (after the gather below)
    auto each_key = [&](auto f) {
        if (flat) {
            for (unsigned sidx = tid; sidx < (unsigned)G * pitch; sidx += MERGE_NT) {
                const unsigned g = sidx / (unsigned)pitch, i = sidx - g * (unsigned)pitch;
                if (i < fcnt[g]) f(lists[sidx]);
            }
        }
        for (int g = tid; g < G && !flat; g += MERGE_NT) {
            const unsigned c = min(counts[g], (unsigned)pitch);
            const uint64_t *l = lists + (size_t)g * pitch;
            for (unsigned i = 0; i < c; i += 8) {  // eight loads in flight before the first use
                uint64_t k[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) k[u] = (i + u < c) ? l[i + u] : 0;
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (i + u < c) f(k[u]);
            }
        }
        if (both) {
            for (int g = 0; g < GA; ++g) {
                const unsigned c = min(countsA[g], (unsigned)pitchA);
                for (unsigned i = tid; i < c; i += MERGE_NT) f(listsA[(size_t)g * pitchA + i]);
            }
        }
    };

    auto index_of = [&](uint32_t pos) -> uint32_t {
        if (!ids) return pos;
        return ((int64_t)pos < n_ids) ? ids[pos] : 0xffffffffu;
    };

    // Gather, region by region.
    if (tid == 0) { lcnt = 0; ccnt = 0; all_or = 0ull; all_and = ~0ull; }
    for (int i = tid; i < 256; i += MERGE_NT) sc.hist[i] = 0;
    __syncthreads();
    // Histogram bits.  Integer distances: the distance byte itself, counted while gathering.
    // Float distances: the eight most significant bits in which the keys differ at all (the
    // bits above them agree), found from the OR and the AND of all keys, counted afterwards.
    constexpr bool ADAPT = sizeof(DistT) != 1;
    unsigned long long my_or = 0ull, my_and = ~0ull;
    auto take = [&](uint64_t k) {
        const unsigned slot = atomicAdd(&lcnt, 1u);
        if (slot < (unsigned)MERGE_CAP) lkeys[slot] = k;
        if constexpr (ADAPT) {
            my_or |= k;
            my_and &= k;
        } else {
            atomicAdd(&sc.hist[(unsigned)(k >> 32) & 255u], 1u);
        }
    };
    unsigned mycnt[MERGE_WG_PER_THREAD];
    if (flat) {
        for (int g = tid; g < G; g += MERGE_NT) fcnt[g] = min(counts[g], (unsigned)pitch);
        __syncthreads();
        for (unsigned sidx = tid; sidx < (unsigned)G * pitch; sidx += MERGE_NT) {
            const unsigned g = sidx / (unsigned)pitch, i = sidx - g * (unsigned)pitch;
            if (i < fcnt[g]) take(lists[sidx]);
        }
    } else {
#pragma unroll
        for (int t = 0; t < MERGE_WG_PER_THREAD; ++t) {
            const int g = tid + t * MERGE_NT;
            mycnt[t] = 0;
            if (g < G) {
                // count and first key fetched together: most regions hold zero or one key
                const unsigned c = min(counts[g], (unsigned)pitch);
                const uint64_t *l = lists + (size_t)g * pitch;
                const uint64_t k0 = l[0];
                mycnt[t] = c;
                if (c) take(k0);
                for (unsigned i = 1; i < c; i += 4) {  // four loads in flight
                    uint64_t k[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) k[u] = (i + u < c) ? l[i + u] : 0;
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (i + u < c) take(k[u]);
                }
            }
        }
        for (int g = tid + MERGE_WG_PER_THREAD * MERGE_NT; g < G; g += MERGE_NT) {  // very wide grids
            const unsigned c = min(counts[g], (unsigned)pitch);
            for (unsigned i = 0; i < c; ++i) take(lists[(size_t)g * pitch + i]);
        }
    }
    if (both) {  // region A on top of region B (few regions, spread over the whole workgroup)
        for (int g = 0; g < GA; ++g) {
            const unsigned c = min(countsA[g], (unsigned)pitchA);
            for (unsigned i = tid; i < c; i += MERGE_NT) take(listsA[(size_t)g * pitchA + i]);
        }
    }
    if constexpr (ADAPT) {
        if (my_or != 0ull || my_and != ~0ull) {
            atomicOr(&all_or, my_or);
            atomicAnd(&all_and, my_and);
        }
    }
    __syncthreads();
    unsigned total = lcnt;
    need = min(need, total);
    bool in_lds = total <= (unsigned)MERGE_CAP;
    if constexpr (!ADAPT) {
        // More keys than LDS holds (loose bounds, many regions): the histogram counted all of them, so
        // the bin of the need-th key is known, and only the keys up to that bin are gathered again.
        if (!in_lds && need > 0) {  // uniform
            select_bin(&sc, need);
            __syncthreads();
            const unsigned bin = sc.bin;
            const unsigned upto = need - sc.need + sc.hist[bin];  // keys in the bins up to `bin`
            __syncthreads();
            if (upto <= (unsigned)MERGE_CAP) {
                if (tid == 0) lcnt = 0;
                __syncthreads();
                each_key([&](uint64_t k) {
                    if (((unsigned)(k >> 32) & 255u) <= bin) lkeys[atomicAdd(&lcnt, 1u)] = k;
                });
                __syncthreads();
                total = upto;
                in_lds = true;
            }
        }
    }
    int TOP = 32;
    if constexpr (ADAPT) {
        const unsigned long long diff = all_or ^ all_and;
        const int top = diff ? 63 - __clzll((long long)diff) : 7;
        TOP = top > 7 ? top - 7 : 0;
        if (in_lds)
            for (unsigned i = tid; i < total; i += MERGE_NT)
                atomicAdd(&sc.hist[(unsigned)(lkeys[i] >> TOP) & 255u], 1u);
        __syncthreads();
    }

    bool done = false;
    if (need > 0 && in_lds) {
        // bin of the need-th key by its most significant byte, and the keys up to that bin
        select_bin(&sc, need);
        __syncthreads();
        const unsigned bin = sc.bin;
        for (unsigned i = tid; i < total; i += MERGE_NT) {
            const uint64_t k = lkeys[i];
            if (((unsigned)(k >> TOP) & 255u) <= bin) {
                const unsigned slot = atomicAdd(&ccnt, 1u);
                if (slot < (unsigned)MERGE_NT) cand[slot] = k;
            }
        }
        __syncthreads();
        const unsigned nc = ccnt;
        if (nc <= (unsigned)MERGE_NT) {  // uniform: rank the candidates against each other
            if ((unsigned)tid < nc) {
                const uint64_t k = cand[tid];
                unsigned rank = 0;
                for (unsigned j = 0; j < nc; ++j) rank += (cand[j] < k) ? 1u : 0u;
                if (rank < need) {
                    DistT d;
                    if constexpr (sizeof(DistT) == 1) d = (DistT)((k >> 32) & 0xff);
                    else d = ord2f((unsigned)(k >> 32));
                    out_idx[(size_t)q * R + rank] = index_of((uint32_t)k);
                    out_dist[(size_t)q * R + rank] = d;
                }
            }
            done = true;
        }
        __syncthreads();
    }

    if (need > 0 && !done) {
        // full radix select, then order the winners by rank
        uint64_t kth;
        if (in_lds) kth = block_radix_select<uint64_t, KBYTES>(lkeys, total, need, &sc);
        else kth = block_radix_select_each<uint64_t, KBYTES>(each_key, need, &sc);
        __syncthreads();
        uint64_t mine[MERGE_CAP / MERGE_NT];
        if (in_lds) {
#pragma unroll
            for (int t = 0; t < MERGE_CAP / MERGE_NT; ++t) {
                const unsigned i = tid + t * MERGE_NT;
                mine[t] = (i < total) ? lkeys[i] : ~0ull;
            }
        }
        if (tid == 0) lcnt = 0;
        __syncthreads();
        if (in_lds) {
#pragma unroll
            for (int t = 0; t < MERGE_CAP / MERGE_NT; ++t) {
                const unsigned i = tid + t * MERGE_NT;
                const bool ok = (i < total) && mine[t] <= kth;
                const unsigned slot = wave_append_slot(ok, &lcnt);
                if (ok) lkeys[slot] = mine[t];
            }
        } else {
            each_key([&](uint64_t k) {
                if (k <= kth) lkeys[atomicAdd(&lcnt, 1u)] = k;  // exactly `need` keys: they are unique
            });
        }
        __syncthreads();
        for (unsigned i = tid; i < need; i += MERGE_NT) {
            const uint64_t k = lkeys[i];
            unsigned rank = 0;
            for (unsigned j = 0; j < need; ++j) rank += (lkeys[j] < k) ? 1u : 0u;
            DistT d;
            if constexpr (sizeof(DistT) == 1) d = (DistT)((k >> 32) & 0xff);
            else d = ord2f((unsigned)(k >> 32));
            out_idx[(size_t)q * R + rank] = index_of((uint32_t)k);
            out_dist[(size_t)q * R + rank] = d;
        }
    }
    for (unsigned i = need + tid; i < (unsigned)R; i += MERGE_NT) {
        out_idx[(size_t)q * R + i] = 0xffffffffu;
        out_dist[(size_t)q * R + i] = pad_dist;
    }

    // Leave every word this call wrote in the workspace zero again, so that the next call
    // finds clean control blocks wherever its own layout puts them.
    if (flat) {
        for (unsigned sidx = tid; sidx < (unsigned)G * pitch; sidx += MERGE_NT) {
            const unsigned g = sidx / (unsigned)pitch, i = sidx - g * (unsigned)pitch;
            if (i < fcnt[g]) lists[sidx] = 0;
        }
        for (int g = tid; g < G; g += MERGE_NT)
            if (fcnt[g]) counts[g] = 0;
    } else {
#pragma unroll
        for (int t = 0; t < MERGE_WG_PER_THREAD; ++t) {
            const int g = tid + t * MERGE_NT;
            if (g < G && mycnt[t]) {
                for (unsigned i = 0; i < mycnt[t]; ++i) lists[(size_t)g * pitch + i] = 0;
                counts[g] = 0;
            }
        }
        for (int g = tid + MERGE_WG_PER_THREAD * MERGE_NT; g < G; g += MERGE_NT) {
            const unsigned c = min(counts[g], (unsigned)pitch);
            for (unsigned i = 0; i < c; ++i) lists[(size_t)g * pitch + i] = 0;
            if (c) counts[g] = 0;
        }
    }
    if (redone || both) {  // the abandoned report of the tiled kernel, or the second half of the result
        __syncthreads();  // (both: every thread is done reading region A)
        for (int g = 0; g < GA; ++g) {
            const unsigned c = min(countsA[g], (unsigned)pitchA);
            for (unsigned i = tid; i < c; i += MERGE_NT) listsA[(size_t)g * pitchA + i] = 0;
        }
        __syncthreads();
        for (int g = tid; g < GA; g += MERGE_NT) countsA[g] = 0;
        if (tid == 0) flags[q] = 0;
    }
    unsigned *z = reinterpret_cast<unsigned *>(hdr);
    for (int i = tid; i < (int)(sizeof(ScanHeader) / 4); i += MERGE_NT) z[i] = 0;
}

constexpr int MERGE_PER = MERGE_CAP / MERGE_NT;
constexpr int MERGE_GU = 4;       // regions per thread whose counts are requested together
constexpr int MERGE_REP = 16;    // replicas of the histogram of a flat gather (in the memory of lkeys)
constexpr int MERGE_SLOTS = 25;   // key slots per thread up to which every slot is visited at once (256 regions of 100)
constexpr int MERGE_GATHER_R = 128, MERGE_GATHER_MIN_R = 32;

// The same for calls whose keys are in one region set (no flags) and many for their number of regions, or whose
// keys are 64 bits of distance and index; R <= MERGE_GATHER_R.  Bound by latency: one workgroup, a chain of round
// trips to memory written by other XCDs.  So the counts of all regions travel at once, and then all keys at once.
// flat: regions that are mostly full (short databases without a sampled bound; the few workgroups of an
// inverted-index query): a slot of a region per thread and register, thousands of keys in a few bins counted in 16
// replicas of the histogram.  Else the places of the keys are laid out in LDS first, from running sums of the
// counts.  Against the kernel above: 14.1 / 20.7 us for one inverted-index query (192 regions of up to 100 keys),
// 10.7 / 14.8 us for 16 queries over 98 regions, 9.6 / 18.7 us for a float scan of 50 M codes (1024 regions).  (Code
// size counts: a second unrolled walk over the 25 slots in the rarely taken part cost every call 3 to 5 us.)
template <typename DistT, int KBYTES, bool FLAT>
__global__ __launch_bounds__(MERGE_NT) void merge_gather_kernel(
    char *__restrict__ ws, size_t ws_stride, size_t counts_off, size_t lists_off, int G,
    unsigned need, int R, DistT pad_dist, uint32_t *__restrict__ out_idx,
    DistT *__restrict__ out_dist, const uint32_t *__restrict__ ids, int64_t n_ids)
{
    // need = min(R, number of codes scanned): at least that many keys were reported.
    // ids: the keys' low words are storage positions and out_idx gets ids[position] (inverted index).
    __shared__ uint64_t lkeys[MERGE_CAP];  // the places of the keys, or the histogram's replicas; then the winners
    __shared__ uint64_t cand[MERGE_NT];
    __shared__ SelectScratch sc;
    __shared__ unsigned lcnt, ccnt;
    __shared__ unsigned long long all_or, all_and;
    __shared__ unsigned rank_s[MERGE_NT / 2];
    __shared__ unsigned fcnt[MERGE_FLAT_G];

    const int tid = threadIdx.x;
    const int q = blockIdx.x;
    ScanHeader *hdr = reinterpret_cast<ScanHeader *>(ws + (size_t)q * ws_stride);
    unsigned *counts = reinterpret_cast<unsigned *>(ws + (size_t)q * ws_stride + counts_off);
    uint64_t *lists = reinterpret_cast<uint64_t *>(ws + (size_t)q * ws_stride + lists_off);
    const int pitch = R;
    const unsigned slots = (unsigned)G * (unsigned)R;
    // every reported key, spread over the threads by region (only where too many of them tie for LDS to hold them)
    auto each_key = [&](auto f) {
        constexpr int step = FLAT ? MERGE_NT / WAVE : MERGE_NT;  // few regions: a wavefront per region
        const unsigned i0 = FLAT ? tid % WAVE : 0, di = FLAT ? WAVE : 1;
        for (int g = FLAT ? tid / WAVE : tid; g < G; g += step) {
            const unsigned c = min(counts[g], (unsigned)pitch);
            const uint64_t *l = lists + (size_t)g * pitch;
            for (unsigned i = i0; i < c; i += 4 * di) {  // four loads in flight before the first use
                uint64_t k[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) k[u] = (i + u * di < c) ? l[i + u * di] : 0;
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (i + u * di < c) f(k[u]);
            }
        }
    };

    auto index_of = [&](uint32_t pos) -> uint32_t {
        if (!ids) return pos;
        return ((int64_t)pos < n_ids) ? ids[pos] : 0xffffffffu;
    };

    if (tid == 0) { lcnt = 0; ccnt = 0; all_or = 0ull; all_and = ~0ull; }
    for (int i = tid; i < 256; i += MERGE_NT) sc.hist[i] = 0;
    for (int i = tid; i < MERGE_NT / 2; i += MERGE_NT) rank_s[i] = 0;
    __syncthreads();
    // Histogram bits.  Integer distances: the distance byte itself.  Float distances: the eight most
    // significant bits in which the keys differ at all (the bits above them agree), found from the OR and the
    // AND of all keys.
    constexpr bool ADAPT = sizeof(DistT) != 1;
    static_assert(FLAT || ADAPT, "byte sums are gathered from filled regions only");
    constexpr int PER = FLAT ? MERGE_SLOTS : MERGE_PER;
    const int lane = lane_id();
    uint64_t key[PER];            // flat: the keys of this thread's slots, ~0 for none
    unsigned place[PER];          // else: where the keys of this thread lie
    unsigned total;
    bool placed = false;          // place[] is set
    // Thousands of keys that differ in a few bins would queue at the same LDS words: 16 replicas, a word apart.
    unsigned *rep = reinterpret_cast<unsigned *>(lkeys);
    static_assert(MERGE_REP * 257 * sizeof(unsigned) <= sizeof(lkeys), "replicas of the histogram");
    auto count = [&](unsigned bin) { atomicAdd(FLAT ? &rep[(lane % MERGE_REP) * 257 + bin] : &sc.hist[bin], 1u); };
    auto join_counts = [&]() {  // the whole workgroup, after a barrier
        if (FLAT && tid < 256) {
            unsigned h = 0;
#pragma unroll
            for (int r = 0; r < MERGE_REP; ++r) h += rep[r * 257 + tid];
            sc.hist[tid] = h;
        }
    };
    if constexpr (FLAT) {
        for (int i = tid; i < MERGE_REP * 257; i += MERGE_NT) rep[i] = 0;
        if (tid < MERGE_FLAT_G) {
            const unsigned c = tid < G ? min(counts[tid], (unsigned)pitch) : 0u;
            fcnt[tid] = c;
            unsigned sum = c;
#pragma unroll
            for (int w = 32; w >= 1; w >>= 1) sum += __shfl_xor(sum, w);
            if (lane == 0 && sum) atomicAdd(&lcnt, sum);
        }
        __syncthreads();
        total = lcnt;
#pragma unroll
        for (int t = 0; t < MERGE_SLOTS; ++t) {
            key[t] = ~0ull;
            if ((unsigned)(t * MERGE_NT) >= slots) continue;  // uniform
            const unsigned s = tid + t * MERGE_NT;
            const unsigned g = s / (unsigned)pitch;
            if (s < slots && s - g * (unsigned)pitch < fcnt[g]) key[t] = lists[s];
        }
    } else {
        // running sums over the wavefront, one atomic per wavefront (the order of the keys does not matter)
        for (int g0 = 0; g0 < G; g0 += MERGE_GU * MERGE_NT) {  // uniform
            unsigned c[MERGE_GU], sum = 0;
#pragma unroll
            for (int u = 0; u < MERGE_GU; ++u) {
                const int g = g0 + u * MERGE_NT + tid;
                c[u] = g < G ? counts[g] : 0u;
            }
#pragma unroll
            for (int u = 0; u < MERGE_GU; ++u) {
                c[u] = min(c[u], (unsigned)pitch);
                sum += c[u];
            }
            const unsigned inc = wave_running_sum(sum);
            unsigned base = 0;
            if (lane == WAVE - 1 && inc > 0) base = atomicAdd(&lcnt, inc);
            unsigned at = lane_value(base, WAVE - 1) + inc - sum;
#pragma unroll
            for (int u = 0; u < MERGE_GU; ++u) {
                const unsigned first = (unsigned)(g0 + u * MERGE_NT + tid) * (unsigned)pitch;
                for (unsigned i = 0; i < c[u] && at + i < (unsigned)MERGE_CAP; ++i) lkeys[at + i] = first + i;
                at += c[u];
            }
        }
        __syncthreads();
        total = lcnt;
        if (total <= (unsigned)MERGE_CAP) {  // uniform
            placed = true;
#pragma unroll
            for (int t = 0; t < MERGE_PER; ++t) {
                const unsigned i = tid + t * MERGE_NT;
                place[t] = i < total ? (unsigned)lkeys[i] : NO_KEY;
            }
#pragma unroll
            for (int t = 0; t < MERGE_PER; ++t) key[t] = place[t] != NO_KEY ? lists[place[t]] : ~0ull;
        }
    }
    const bool in_regs = FLAT || placed;               // key[] is set
    auto own_keys = [&](auto f) {
        if (!in_regs) return;  // uniform
#pragma unroll
        for (int t = 0; t < PER; ++t) {
            if ((unsigned)(t * MERGE_NT) >= (FLAT ? slots : total)) break;  // uniform
            if (key[t] != ~0ull) f(key[t]);
        }
    };
    if constexpr (ADAPT) {
        unsigned long long my_or = 0ull, my_and = ~0ull;
        own_keys([&](uint64_t k) { my_or |= k; my_and &= k; });
#pragma unroll
        for (int w = 32; w >= 1; w >>= 1) {
            my_or |= __shfl_xor(my_or, w);
            my_and &= __shfl_xor(my_and, w);
        }
        if (lane == 0 && (my_or != 0ull || my_and != ~0ull)) {
            atomicOr(&all_or, my_or);
            atomicAnd(&all_and, my_and);
        }
    } else {
        own_keys([&](uint64_t k) { count((unsigned)(k >> 32) & 255u); });
        __syncthreads();
        join_counts();
    }
    __syncthreads();
    need = min(need, total);
    int TOP = 32;
    if constexpr (ADAPT) {
        const unsigned long long diff = all_or ^ all_and;
        const int top = diff ? 63 - __clzll((long long)diff) : 7;
        TOP = top > 7 ? top - 7 : 0;
        own_keys([&](uint64_t k) { count((unsigned)(k >> TOP) & 255u); });
        __syncthreads();
        join_counts();
        __syncthreads();
    }

    bool done = false;
    if (need > 0 && in_regs) {  // uniform
        // bin of the need-th key by its most significant byte, and the keys up to that bin
        select_bin(&sc, need);
        __syncthreads();
        const unsigned bin = sc.bin;
        auto keep = [&](uint64_t k) {
            if (((unsigned)(k >> TOP) & 255u) <= bin) {
                const unsigned slot = atomicAdd(&ccnt, 1u);
                if (slot < (unsigned)MERGE_NT) cand[slot] = k;
            }
        };
        own_keys(keep);
        __syncthreads();
        const unsigned nc = ccnt;
        if (nc <= (unsigned)MERGE_NT) {  // uniform: rank the candidates against each other
            // each candidate's comparisons are split over as many threads as there are to go round
            const unsigned span = nc <= 128u ? 128u : nc <= 256u ? 256u : nc <= 512u ? 512u : 1024u;
            const unsigned parts = MERGE_NT / span, e = tid & (span - 1u), p = tid / span;
            uint64_t k = ~0ull;
            unsigned rank = 0;
            if (e < nc) {
                k = cand[e];
                const unsigned hi = nc * (p + 1u) / parts;
#pragma unroll 4
                for (unsigned j = nc * p / parts; j < hi; ++j) rank += (cand[j] < k) ? 1u : 0u;
                if (parts > 1u) atomicAdd(&rank_s[e], rank);  // uniform
            }
            __syncthreads();
            if ((unsigned)tid < nc) {
                if (parts > 1u) rank = rank_s[tid];
                if (rank < need) {
                    DistT d;
                    if constexpr (sizeof(DistT) == 1) d = (DistT)((k >> 32) & 0xff);
                    else d = ord2f((unsigned)(k >> 32));
                    out_idx[(size_t)q * R + rank] = index_of((uint32_t)k);
                    out_dist[(size_t)q * R + rank] = d;
                }
            }
            done = true;
        }
        __syncthreads();
    }

    if (need > 0 && !done) {
        // full radix select, then order the winners by rank
        const unsigned held = FLAT ? slots : total;  // key[t] of thread tid is number tid + t MERGE_NT of these
        if (held <= (unsigned)MERGE_CAP) {           // uniform
            constexpr int HELD = PER < MERGE_PER ? PER : MERGE_PER;
#pragma unroll
            for (int t = 0; t < HELD; ++t)
                if (tid + t * MERGE_NT < held) lkeys[tid + t * MERGE_NT] = key[t];  // (an empty slot's ~0 comes last)
            __syncthreads();
            const uint64_t kth = block_radix_select<uint64_t, KBYTES>(lkeys, held, need, &sc);
            __syncthreads();
            if (tid == 0) lcnt = 0;
            __syncthreads();
#pragma unroll
            for (int t = 0; t < HELD; ++t)
                if (tid + t * MERGE_NT < held && key[t] <= kth) lkeys[atomicAdd(&lcnt, 1u)] = key[t];  // exactly `need`
        } else {
            const uint64_t kth = block_radix_select_each<uint64_t, KBYTES>(each_key, need, &sc);
            __syncthreads();
            if (tid == 0) lcnt = 0;
            __syncthreads();
            each_key([&](uint64_t k) {
                if (k <= kth) lkeys[atomicAdd(&lcnt, 1u)] = k;  // exactly `need` keys: they are unique
            });
        }
        __syncthreads();
        for (unsigned i = tid; i < need; i += MERGE_NT) {
            const uint64_t k = lkeys[i];
            unsigned rank = 0;
            for (unsigned j = 0; j < need; ++j) rank += (lkeys[j] < k) ? 1u : 0u;
            DistT d;
            if constexpr (sizeof(DistT) == 1) d = (DistT)((k >> 32) & 0xff);
            else d = ord2f((unsigned)(k >> 32));
            out_idx[(size_t)q * R + rank] = index_of((uint32_t)k);
            out_dist[(size_t)q * R + rank] = d;
        }
    }
    for (unsigned i = need + tid; i < (unsigned)R; i += MERGE_NT) {
        out_idx[(size_t)q * R + i] = 0xffffffffu;
        out_dist[(size_t)q * R + i] = pad_dist;
    }

    // Leave every word this call wrote in the workspace zero again, so that the next call
    // finds clean control blocks wherever its own layout puts them.
    if constexpr (FLAT) {
#pragma unroll
        for (int t = 0; t < MERGE_SLOTS; ++t)
            if (key[t] != ~0ull) lists[tid + t * MERGE_NT] = 0;
    } else if (placed) {
#pragma unroll
        for (int t = 0; t < MERGE_PER; ++t)
            if (place[t] != NO_KEY) lists[place[t]] = 0;
    } else {
        for (int g = tid; g < G; g += MERGE_NT) {
            const unsigned c = min(counts[g], (unsigned)pitch);
            for (unsigned i = 0; i < c; ++i) lists[(size_t)g * pitch + i] = 0;
        }
        __syncthreads();
    }
    for (int g = tid; g < G; g += MERGE_NT) counts[g] = 0;
    unsigned *z = reinterpret_cast<unsigned *>(hdr);
    for (int i = tid; i < (int)(sizeof(ScanHeader) / 4); i += MERGE_NT) z[i] = 0;
}

// What the single-query kernels leave in a region of region B.
enum MergeFill {
    MERGE_SPARSE,  // a key or two: a sampled bound stood before the scan
    MERGE_MIXED,   // anything (batches over an inverted index)
    MERGE_FILLED   // mostly R keys: no sampled bound, or the few long workgroups of an inverted-index query
};

// One merge workgroup per query.  The gathering kernel takes filled regions whose slots fit its registers, and float
// keys behind a sampled bound; not where hardly a key is there to gather.  us per call, the kernel above / gathering:
//   byte sums, 16 queries x 100 k codes, m = 16 (98 regions): R = 1 13.0 / 13.9, R = 20 15.4 / 15.6, R = 100 24.9 / 20.3;
//   floats, one query, 4-bit components, m = 16: 20 k codes (20 regions) R = 1 13.3 / 14.4, R = 10 17.2 / 14.9, 100 k R = 1
//   16.0 / 14.6; behind a bound, 2 M codes: R = 1 21.5 / 23.1, R = 20 26.7 / 26.9, R = 50 27.6 / 26.6, R = 100 30.1 / 27.3.
// Visiting every slot of sparse regions (256 regions, R = 100) took calls of 5 to 7 queries 8 us of 28.
template <typename DistT, int KBYTES>
inline int launch_merge(int nq, hipStream_t st, MergeFill fill, char *ws, size_t ws_stride, size_t counts_off,
                        size_t lists_off, int G, unsigned need, int R, DistT pad_dist, uint32_t *out_idx, DistT *out_dist,
                        size_t countsA_off, size_t listsA_off, int GA, int pitchA, unsigned *flags, const uint32_t *ids,
                        int64_t n_ids)
{
    constexpr bool BYTES = sizeof(DistT) == 1;
    const int64_t slots = (int64_t)G * R;
    if (!flags && R <= MERGE_GATHER_R) {
        if (fill == MERGE_FILLED && G <= MERGE_FLAT_G && slots <= MERGE_SLOTS * MERGE_NT && (BYTES ? slots >= 2048 : R >= 64 || (G >= 8 && slots >= 96))) {
            launch(QADC_PROF_MERGE, (merge_gather_kernel<DistT, KBYTES, true>), dim3(nq), dim3(MERGE_NT), 0, st, ws,
                   ws_stride, counts_off, lists_off, G, need, R, pad_dist, out_idx, out_dist, ids, n_ids);
            return QADC_OK;
        }
        if constexpr (!BYTES) {
            if (fill == MERGE_SPARSE && R >= MERGE_GATHER_MIN_R) {
                launch(QADC_PROF_MERGE, (merge_gather_kernel<DistT, KBYTES, false>), dim3(nq), dim3(MERGE_NT), 0, st, ws,
                       ws_stride, counts_off, lists_off, G, need, R, pad_dist, out_idx, out_dist, ids, n_ids);
                return QADC_OK;
            }
        }
    }
#define QADC_MERGE(VISIT_)                                                                                             \
    launch(QADC_PROF_MERGE, (merge_topk_kernel<DistT, KBYTES, VISIT_>), dim3(nq), dim3(MERGE_NT), 0, st, ws, ws_stride, \
           counts_off, lists_off, G, need, R, pad_dist, out_idx, out_dist, countsA_off, listsA_off, GA, pitchA, flags,  \
           ids, n_ids)
    if constexpr (BYTES) {
        if (fill == MERGE_SPARSE && !flags) {
            QADC_MERGE(false);
            return QADC_OK;
        }
    }
    QADC_MERGE(true);
#undef QADC_MERGE
    return QADC_OK;
}

// Workspace layout of one scan call: per query a ScanHeader, counts[G], lists[G][R].
struct ScanLayout {
    size_t counts_off, lists_off, stride;
};

inline ScanLayout scan_layout(int G, int R)
{
    ScanLayout l;
    l.counts_off = sizeof(ScanHeader);
    l.lists_off = l.counts_off + align_up((size_t)G * sizeof(unsigned), 256);
    l.stride = l.lists_off + align_up((size_t)G * R * sizeof(uint64_t), 256);
    return l;
}

// Queries per launch so that the workspace stays within 256 MiB.
inline int scan_query_batch(size_t stride, int nq)
{
    int64_t qb = (int64_t)((256ull << 20) / stride);
    if (qb < 1) qb = 1;
    if (qb > nq) qb = nq;
    if (qb > 65535) qb = 65535;
    return (int)qb;
}

// Tuning knobs: the QADC_* environment variables.  They change launch shapes and which of the
// equivalent kernels runs, never a result.  An entry point reads them ONCE, when it is called
// (knobs_refresh), into the calling thread's copy; everything below it uses that copy.  -1: not set.
struct Knobs {
    int scan_nt, scan_wgs, seed_min_tiles, seed_wgs, tiled, tiled_seed, scan_f32_wgs;
    int tiled_mfma, tiled_decoded, mfma_min_q, mfma_min_q2, mfma_min_q4, mfma_waves;
    int ivf_wgs, ivf_seed, ivf_units, ivf_seed_parts, ivf_shared, ivf_shared_wgs, ivf_shared_min_pairs, ivf_seed_probes,
        ivf_wide_q;
};
const Knobs &knobs();
void knobs_refresh();
inline int knob_or(int value, int dflt) { return value >= 0 ? value : dflt; }

}  // namespace qadc
