// What the Index step's filter (qadc_ivf_filter.hip) and the selection from its bounds (qadc_ivf.hip) share: where the bounds
// of a query lie, which cells a bound is of, and the filter's entry points.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include "qadc_common.h"

namespace qadc {

// Where the bounds of query i lie: in its own row of K distances, which the selection may overwrite.
__host__ __device__ inline uint16_t *ivf_filter_row(float *dist, int K, size_t i)
{
    return reinterpret_cast<uint16_t *>((reinterpret_cast<uintptr_t>(dist + i * (size_t)K) + 15) & ~(uintptr_t)15);
}

// A tile of 32 cells has eight bounds; number `half`, k of them (half < 2, k < 4) lies at place 8 tile + 4 half + k of the row and
// is of the four cells from 32 tile + 8 k + 4 half on.
__host__ __device__ inline int ivf_filter_place(int tile, int half, int k) { return 8 * tile + 4 * half + k; }
__host__ __device__ inline unsigned ivf_filter_first_cell(unsigned place)
{
    return (place >> 3) * 32u + (place & 3u) * 8u + ((place >> 2) & 1u) * 4u;
}

size_t ivf_filter_bytes(int K, int d, int nq);
bool ivf_filter_pays(int K, int d, int nq, int nprobe);
void ivf_filter_convert(const float *coarse, int K, int d, const float *queries, int nq, void *room, hipStream_t st);
const float2 *ivf_filter(int K, int d, int nq, int i0, int ni, void *room, float *dist, int *components, unsigned **rest,
                         hipStream_t st);

}  // namespace qadc
