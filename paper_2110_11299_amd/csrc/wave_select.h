// Wavefront-level primitives shared by the kernels: reductions and scans without LDS, the
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
// (every lane has a source, so that what stands in for a missing one does not matter; with 0 the compiler makes one instruction of the
// move and what is done with it)
template <int CTRL> __device__ __forceinline__ int dpp_move(int x)
{
    return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xF, 0xF, true);
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

// x of the even and of the odd row of 16 in every pair of rows, and of the lower and the upper 32 lanes: both in all lanes.
// v_permlane16_swap exchanges the odd rows of its first operand with the even ones of its second, v_permlane32_swap the upper half of
// the first with the lower half of the second.
struct Halves { int lower, upper; };
__device__ __forceinline__ Halves row_halves(int x)
{
    const auto s = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)x, false, false);
    return Halves{(int)s[0], (int)s[1]};
}
__device__ __forceinline__ Halves wave_halves(int x)
{
    const auto s = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)x, false, false);
    return Halves{(int)s[0], (int)s[1]};
}

// Exclusive prefix and total of a per-lane count over the four lanes (c, 0..3) of a unit, in lane
// order g = 0..3.
__device__ __forceinline__ int unit_excl_scan(int x, int g, int *total)
{
    const Halves a = row_halves(x), b = wave_halves(a.lower + a.upper);
    *total = b.lower + b.upper;
    return ((g & 1) ? a.lower : 0) + ((g & 2) ? b.lower : 0);
}

// x from the lane that differs in bit log2(OFF) of its number; for OFF = 4 from the mirror image in the lane's 8 (which lies in the
// other half of them: as good where all 8 are summed).
template <int OFF> __device__ __forceinline__ float other_half(float x)
{
    static_assert(OFF == 1 || OFF == 2 || OFF == 4 || OFF == 8, "DPP reaches a row of 16 lanes");
    constexpr int CTRL = OFF == 1 ? kDppXor1 : OFF == 2 ? kDppXor2 : OFF == 4 ? kDppHalfMirror : 0x128 /* row_ror:8 */;
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}
// Lanes whose bit log2(OFF) is clear get x summed over both halves, the others y.  v_permlane32_swap exchanges the upper half of
// x with the lower half of y, v_permlane16_swap the odd rows of 16 of x with the even ones of y.
template <int OFF> __device__ __forceinline__ float halves_sum(float x, float y, int lane)
{
    if constexpr (OFF >= 16) {
        const unsigned a = __float_as_uint(x), b = __float_as_uint(y);
        const auto s = OFF == 32 ? __builtin_amdgcn_permlane32_swap(a, b, false, false) : __builtin_amdgcn_permlane16_swap(a, b, false, false);
        return __uint_as_float(s[0]) + __uint_as_float(s[1]);
    } else {
        const float sx = x + other_half<OFF>(x), sy = y + other_half<OFF>(y);
        return (lane & OFF) ? sy : sx;
    }
}
// x summed over both halves, in all lanes.
template <int OFF> __device__ __forceinline__ float halves_sum(float x)
{
    if constexpr (OFF >= 16) return halves_sum<OFF>(x, x, 0);
    else return x + other_half<OFF>(x);
}
template <int OFF> __device__ __forceinline__ float halves_max(float x)
{
    if constexpr (OFF >= 16) {
        const unsigned a = __float_as_uint(x);
        const auto s = OFF == 32 ? __builtin_amdgcn_permlane32_swap(a, a, false, false) : __builtin_amdgcn_permlane16_swap(a, a, false, false);
        return fmaxf(__uint_as_float(s[0]), __uint_as_float(s[1]));
    } else {
        return fmaxf(x, other_half<OFF>(x));
    }
}
__device__ __forceinline__ float wave_all_sum(float x)
{
    return halves_sum<32>(halves_sum<16>(halves_sum<8>(halves_sum<4>(halves_sum<2>(halves_sum<1>(x))))));
}
__device__ __forceinline__ float wave_all_max(float x)
{
    return halves_max<32>(halves_max<16>(halves_max<8>(halves_max<4>(halves_max<2>(halves_max<1>(x))))));
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
