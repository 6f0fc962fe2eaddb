// Shared host/device helpers of the Quick ADC HIP library (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <stdarg.h>

#include "qadc.h"

namespace qadc {

// Thread-local message of the last failing call.
char *err_buf();
int fail(int code, const char *fmt, ...);

#define QADC_HIP_TRY(expr)                                                              \
    do {                                                                                \
        hipError_t e_ = (expr);                                                         \
        if (e_ != hipSuccess)                                                           \
            return qadc::fail(QADC_EHIP, "%s: %s", #expr, hipGetErrorString(e_));       \
    } while (0)

constexpr int WAVE = 64;

__device__ __forceinline__ int lane_id() { return (int)__lane_id(); }

// Number of set bits of `m` below this lane.
__device__ __forceinline__ unsigned rank_in_mask(unsigned long long m)
{
    return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                     __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

// Values of other lanes of the wavefront without a trip through LDS (a __shfl takes some hundred cycles, these four to eight
// each; the kernels of a single query are chains of such steps: 10 M codes 32.0 -> 30.5 us per call, an inverted
// index of 100 M 60.7 -> 58.5).
// All 64 lanes take part.  DPP controls: quad_perm 1 0 3 2 = 0xB1, 2 3 0 1 = 0x4E, 3 2 1 0 = 0x1B, row_shr n = 0x110 + n,
// row_ror 8 = 0x128, row_half_mirror = 0x141, row_bcast 15 / 31 (last lane of a row of 16, of the first 32, to the rows behind) =
// 0x142 / 0x143.
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ unsigned dpp_or_zero(unsigned v)
{
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
}
// inclusive running sum over the lanes
__device__ __forceinline__ unsigned wave_running_sum(unsigned v)
{
    v += dpp_or_zero<0x111>(v);
    v += dpp_or_zero<0x112>(v);
    v += dpp_or_zero<0x114>(v);
    v += dpp_or_zero<0x118>(v);
    v += dpp_or_zero<0x142, 0xa>(v);
    v += dpp_or_zero<0x143, 0xc>(v);
    return v;
}
// lane l ^ X, X a power of two
template <int X>
__device__ __forceinline__ unsigned lane_xor(unsigned v)
{
    if constexpr (X == 1) return dpp_or_zero<0xB1>(v);
    else if constexpr (X == 2) return dpp_or_zero<0x4E>(v);
    else if constexpr (X == 4) return dpp_or_zero<0x1B>(dpp_or_zero<0x141>(v));  // (7 - l, then 3 - l within four)
    else if constexpr (X == 8) return dpp_or_zero<0x128>(v);
    else return (unsigned)__shfl_xor((int)v, X);
}
// lane `from`'s value, from the same in every lane
__device__ __forceinline__ unsigned lane_value(unsigned v, int from)
{
    return (unsigned)__builtin_amdgcn_readlane((int)v, from);
}

// Wave-aggregated append to an LDS list: lanes with `pred` get distinct slots
// counter .. counter+k-1 with one atomic per wave.  Returns the slot (valid when pred).
__device__ __forceinline__ unsigned wave_append_slot(bool pred, unsigned *counter)
{
    unsigned long long m = __ballot(pred);
    unsigned base = 0;
    if (m == 0) return 0;
    int leader = __ffsll((long long)m) - 1;
    if (lane_id() == leader) base = atomicAdd(counter, (unsigned)__popcll(m));
    base = lane_value(base, leader);
    return base + rank_in_mask(m);
}

static inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
static inline size_t align_up(size_t a, size_t b) { return (a + b - 1) / b * b; }

}  // namespace qadc
