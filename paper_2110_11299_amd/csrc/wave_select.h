// Wavefront-level selection primitives shared by the predictor kernels: DPP reductions and scans, the
// lowest set bits of a word, and the exact int8 score of one (unit, key) pair.  Device code only; everything is
// internal to the translation unit that includes it.
#pragma once

#include "dsa_internal.h"

namespace dsa {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

// Wavefront reductions without LDS traffic: butterfly inside each row of 16 lanes with DPP
// (quad permutes, then the two mirrors), then the four row results through v_readlane into
// scalar registers.  The result is wavefront-uniform and lives in an SGPR.
template <int CTRL> __device__ __forceinline__ int dpp_move(int x)
{
    return __builtin_amdgcn_update_dpp(x, x, CTRL, 0xF, 0xF, false);
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141, kDppMirror = 0x140;

__device__ __forceinline__ int wave_sum(int x)
{
    x += dpp_move<kDppXor1>(x);
    x += dpp_move<kDppXor2>(x);
    x += dpp_move<kDppHalfMirror>(x);
    x += dpp_move<kDppMirror>(x);
    return __builtin_amdgcn_readlane(x, 0) + __builtin_amdgcn_readlane(x, 16) +
           __builtin_amdgcn_readlane(x, 32) + __builtin_amdgcn_readlane(x, 48);
}
// Inclusive prefix sum over the 64 lanes: Hillis-Steele inside each row of 16 lanes with DPP row
// shifts (zero fill), then the totals of the lower rows through v_readlane.  *total = wavefront sum.
__device__ __forceinline__ int wave_incl_scan(int x, int lane, int *total)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, true);   // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, true);   // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, true);   // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, true);   // row_shr:8
    const int t0 = __builtin_amdgcn_readlane(x, 15), t1 = __builtin_amdgcn_readlane(x, 31),
              t2 = __builtin_amdgcn_readlane(x, 47), t3 = __builtin_amdgcn_readlane(x, 63);
    const int row = lane >> 4;
    x += (row >= 1 ? t0 : 0) + (row >= 2 ? t1 : 0) + (row >= 3 ? t2 : 0);
    *total = t0 + t1 + t2 + t3;
    return x;
}

// Exclusive prefix and total of a per-lane count over the four lanes (c, 0..3) of a unit, in lane
// order g = 0..3.
__device__ __forceinline__ int unit_excl_scan(int x, int g, int *total)
{
    const int s1 = __shfl_xor(x, 16, kWave);      // lane g ^ 1
    const int s2 = __shfl_xor(x, 32, kWave);      // lane g ^ 2
    const int s3 = __shfl_xor(s1, 32, kWave);     // lane g ^ 3
    *total = x + s1 + s2 + s3;
    // g ^ 1 < g iff bit 0 of g is set; g ^ 2 < g and g ^ 3 < g iff bit 1 is set
    return ((g & 1) ? s1 : 0) + ((g & 2) ? s2 + s3 : 0);
}

// Makes LDS writes of some lanes of a wavefront visible to reads of its other lanes.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Exact score of (unit, key): sum over the unit's vec rows of the int8 dot product.
__device__ __forceinline__ int unit_key_score(const int *__restrict__ qu, const int8_t *__restrict__ krow,
                                              int vec, int k4)
{
    int s = 0;
    for (int c4 = 0; c4 < k4; c4 += 4) {
        const v4i kk = *reinterpret_cast<const v4i *>(krow + 4 * c4);
        for (int r = 0; r < vec; ++r) {
            const int *q = qu + r * k4 + c4;
            s = __builtin_amdgcn_sdot4(q[0], kk.x, s, false);
            s = __builtin_amdgcn_sdot4(q[1], kk.y, s, false);
            s = __builtin_amdgcn_sdot4(q[2], kk.z, s, false);
            s = __builtin_amdgcn_sdot4(q[3], kk.w, s, false);
        }
    }
    return s;
}

// m with all but its r lowest set bits cleared (r <= 0: none kept).
__device__ __forceinline__ unsigned lowest_set_bits(unsigned m, int r)
{
    if (r <= 0) return 0u;
    if (r >= __popc(m)) return m;
    unsigned rest = m;
    for (int i = 0; i < r; ++i) rest &= rest - 1;
    return m & ~rest;
}

}  // namespace
}  // namespace dsa
