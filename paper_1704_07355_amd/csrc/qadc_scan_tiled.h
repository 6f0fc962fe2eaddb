// Interface of the query-tiled scan (qadc_scan_tiled.hip) towards the scan driver.
#pragma once

#include "qadc_common.h"

namespace qadc {

constexpr int TILED_Q = 8;             // queries per workgroup
// threads per workgroup: with m = 64 (B = 32) one workgroup's tables fill 128 KiB of the LDS,
// so that workgroup is made twice as large to keep enough wavefronts on the CU
constexpr int tiled_nt(int B) { return B >= 32 ? 1024 : 512; }
constexpr int TILED_LCAP = 64;         // keys a workgroup can report per query
constexpr int TILED_MAX_CHUNKS = 1024; // database chunks per query
constexpr int TILED_MFMA_MAX_CHUNKS = 4096;  // the same for small batches on the matrix-core kernel
constexpr int TILED_MIN_Q = 8;         // smallest batch worth tiling
constexpr int TILED_MFMA_MIN_Q = 16;   // smallest batch for the matrix-core kernel in a small workspace (else: mfma_pays)
constexpr int TILED_MFMA_MIN_Q_B4 = 32;  // ... of 4-byte codes, in any workspace
constexpr int TILED_MFMA_MIN_Q2 = 64;  // smallest batch for its 64-queries-per-wavefront form
constexpr int TILED_MFMA_MIN_Q4 = 128; // ... for 128 queries per wavefront (codes of up to 8 bytes)

// Workgroup id -> (query group, database chunk).  Workgroups are handed to the 8 XCDs in turn,
// each XCD with an L2 of its own: XCD x = id % 8 takes the chunks congruent to x, and all query
// groups of a chunk follow each other in its share of the ids, so that the chunk is fetched
// from HBM once and every XCD gets the same mix of groups, whichever of them are active.
__device__ __forceinline__ void tiled_group_and_chunk(int ngroups, int &grp, int &chunk)
{
    const unsigned id = blockIdx.x;
    const unsigned slot = id >> 3;
    grp = (int)(slot % (unsigned)ngroups);
    chunk = (int)((slot / (unsigned)ngroups) * 8u + (id & 7u));
}

struct TiledPlan {
    int B, GC;
    int64_t chunk;
    size_t lds_bytes;
    bool mfma;  // the matrix-core kernel scans the batch
};

// What scan_u8_decoded_kernel needs beside the quantized tables: the codebooks [m][16][d / m] and queries [nq][d] they come from,
// the quantizers' steps [nq], and room (see search_u8).  Null where a caller has only the tables.
struct DecodedBatch {
    const float *codebooks, *queries, *deltas;
    int d;
    char *room;
    size_t room_bytes;
};
bool decoded_pays(int B, int64_t n, int nq, int cap, int R, const DecodedBatch &db);
// Does run_tiled_scan take that route?
bool scans_decoded(const TiledPlan &t, int64_t n, int nq, int cap, int R, const uint8_t *qluts16, const DecodedBatch *decoded);
// The database lies in blocks of `block` codes.  A part of the scan takes codes from .. to - 1 of every block (the last one may end before
// that), in `per_block` units of unit_codes codes; `word`: where their bits start.
constexpr int DECODED_PARTS = 4;
struct DecodedPart {
    int from, to, unit_codes, per_block, units, word;
    unsigned limit;
};
// What it has left: for set s (of `queries` queries) and a part's unit u, bit u % 32 of word s * pitch + word + u / 32; and
// everything behind a part of which more pairs passed (passed[part]) than its limit.  Null: nothing was done.
struct DecodedLeft {
    const unsigned *bits, *passed;
    int64_t n;
    int pitch, queries, nparts, block, blocks;
    DecodedPart parts[DECODED_PARTS];
};
// The codes c0 .. c1 - 1 of a unit (none where c1 <= c0).
__device__ __forceinline__ void decoded_unit(const DecodedLeft &all, const DecodedPart &of, int unit, int64_t &c0, int64_t &c1)
{
    const int z = unit / of.per_block, at = of.from + (unit - z * of.per_block) * of.unit_codes;
    c0 = (int64_t)z * all.block + at;
    c1 = min(all.n, c0 + min(of.unit_codes, of.to - at));
}
// Has it stopped behind one of the first k parts?
__device__ __forceinline__ bool decoded_stopped(const DecodedLeft &all, int k)
{
    for (int i = 0; i < k; ++i)
        if (all.passed[i] > all.parts[i].limit) return true;
    return false;
}
DecodedLeft run_decoded_scan(const TiledPlan &t, const uint8_t *codes, int64_t n, int nq, int cap, int R, const uint8_t *qluts,
                             unsigned *taus, char *ws, size_t ws_stride, size_t countsA_off, size_t listsA_off,
                             unsigned *flags, const DecodedBatch &db, hipStream_t st);

// 4-bit codes of B bytes that the byte-lane kernels scan faster than the matrix-core kernel
bool tiled_bytes_pay(int B, int64_t n, int nq);

// May a batch of 4-bit codes of B bytes go to the matrix-core kernel?  Not where a tuning variable says otherwise.
bool mfma_allowed(int B, int nq);

// codes4: 4-bit codes with the queries' 16-entry tables at hand (what the matrix-core kernel reads), and mfma_allowed
// small: the plan of the scan driver's smaller workspace
bool make_tiled_plan(int64_t n, int m, int nq, bool codes4, bool small, TiledPlan *t);

// tau kernel + tiled scan kernel for `nq` queries whose control blocks (histogram, pair
// tables) were filled by the seed/prepare kernel.  qluts16: the queries' 16-entry quantized
// tables [nq][m][16] when the codes are 4-bit (null for 8-bit components).  Region A of query q: counts at
// ws + q*ws_stride + countsA_off ([GC] u32), lists at + listsA_off ([GC][TILED_LCAP] u64).
int run_tiled_scan(const TiledPlan &t, const uint8_t *codes, int64_t n, int nq, int cap, int R,
                   unsigned *taus, char *ws, size_t ws_stride, size_t countsA_off, size_t listsA_off,
                   unsigned *flags, const uint8_t *qluts16, const DecodedBatch *decoded, hipStream_t st);

// Pair tables of the batch + the sampled histograms behind the bounds, in the query-tiled way:
// what seed_u8_kernel does per query.  `sample_codes`: codes of the sample per query.
int run_tiled_seed(const TiledPlan &t, const uint8_t *codes, int64_t n, const uint8_t *qluts, int nq, int cap,
                   int R, int wide, int64_t sample_codes, char *ws, size_t ws_stride, hipStream_t st);

}  // namespace qadc
