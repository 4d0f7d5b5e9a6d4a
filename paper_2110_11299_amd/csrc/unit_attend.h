// Exact attention of a unit of 8 or 4 query rows that share one list of kept keys (paper section 5.1), by one 64-lane wavefront
// on the bf16 matrix cores.  What attention_units_bf16 and the predictor that goes on to attend share.
// Device code only; everything is internal to the translation unit that includes it.
#pragma once

#include "row_attend.h"

namespace dsa {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// A unit of vec rows (8 or 4) with bfloat16 inputs by one wavefront, in one pass over the unit's keys: key and value rows of a step
// of 32 keys pass through one tile in LDS, the keys first, gathered together and one step ahead, or (DIRECT, below) each in turn.  Scores as in
// attention_groups_bf16, but they stay in the lane that owns them (query c, keys 4g..4g+3 of both tiles), which is where the second
// product wants its weights: neither scores nor weights pass through LDS.  The exponentials are taken relative to a running
// reference that is moved only when a score exceeds it by a factor of 2^kUnitSlack, so that a step needs no reduction across lanes.
// Every list length fits (4 bytes per key and wavefront; 96 KB of LDS with 4096 keys at D = 128).
//
// What bounds it, in the predictor's launch: LDS (8 writes of 14.3 cycles, 4 reads of 4.7 and 8 of 2.8 per step and CU) and vector issue (62 % of the time at
// N = 64, L = 2000, keep = 200, VEC = 4), next to them the latency of list -> gather -> tile for short lists.  By itself (DIRECT): the L1, and the latency of a
// gather that nothing of the same wavefront hides.
// Measured (kernel alone, rows through registers): that shape 213 -> 94 us against one row per wavefront (attention_rows), which gathers the four
// times 3.3 GB; VEC = 8, N = 16, L = 4096, keep = 205: 44.7 -> 29 us, N = 64, L = 2048, keep = 102: 51 -> 35 us, D = 128,
// N = 16, L = 8192, keep = 82: 72.6 -> 55 us against two passes with the scores in LDS.  A key and a value tile side by side
// cost occupancy at D = 128 (59 us); rows padded to 16 bytes more instead of swizzled: 96 us at the first shape.
// The error against 64 bits (two-norm): L = 4096, keep = 205, VEC = 8 4.5e-6, L = 2000, keep = 200, VEC = 4 4.3e-6, D = 128,
// L = 8192, keep = 82, VEC = 8 4.0e-6; 3.7e-4 to 4.2e-4 there with weights of one bf16.
constexpr float kUnitSlack = 16.f;

// Where the 16-byte pieces of tile row r are: piece p at p ^ unit_swizzle(r).  A 16-byte read serves lanes 0-3, 12-15, 20-23 and 24-27
// at once (then the other sixteen, then the upper half the same way), an 8-byte one 32 neighbours: with this the score operand takes
// 4.7 cycles per instruction and the transposing read 2.8, on every bank once, against 8.4 and 4.4 with (r & 3) << 1 | (r >> 2 & 1) (D = 64).
template <int D> __device__ __forceinline__ unsigned unit_swizzle(unsigned r) { return (r & 7u) * (D / 64); }

template <int D> constexpr int unit_tile_bytes() { return 32 * 2 * D; }        // key rows, then value rows

// The unit from its list (key(t): entry t) to its rows of O (both Q and O from the unit's first row on), with a reference that may
// lag the maximum by a factor of 2^slack.  Returns whether every sum was finite.
// DIRECT: the gathered rows go straight to LDS, a tile of keys and then one of values, each requested as soon as the operands of the one before it
// are in registers.  Nothing is on its way while they are waited for, but a KB takes 18 cycles of a CU instead of 25 (L1 and LDS write one after
// the other), and 22 (D = 64) to 38 registers less leave five and four wavefronts per SIMD instead of four and three, which cover for each other.  Kernel by
// itself, through registers and so: D = 64, VEC = 4, N = 64, L = 2000, keep = 200 92 to 94 and 80 to 84 us (by box; up to 23 TB/s of gathers), VEC = 8, N = 16, L = 4096, keep = 205 28.1 and
// 26.7, D = 128, N = 16, L = 8192, keep = 82 55.2 and 48.2, VEC = 4, N = 4, L = 4096, keep = 400 44.0 and 35.3.  In the predictor's launch, whose
// registers leave four wavefronts per SIMD either way, groups of 8 lose (N = 16, L = 4096, keep = 205 44.7 and 49.1 us) and groups of 4 win 2 %: left.
// Tiles for keys and values, one step ahead: occupancy (87.6, 26.6, 70.5 us).
template <int D, bool DIRECT, typename Key>
__device__ __forceinline__ bool unit_rows(const uint16_t *Q, const uint16_t *K, const uint16_t *V, Key &&key, float *O, int vec,
                                          int keep, int keep_pad, float scale, int lane, char *tile, float slack)
{
    constexpr int KS = D / 32, CT = D / 16;
    constexpr int ROW = D * 2;             // bytes of a row in LDS
    constexpr int LPR = D / 8, RPI = kWave / LPR, VP = 32 / RPI;
    const int c = lane & 15, g = lane >> 4;
    unsigned *sl = reinterpret_cast<unsigned *>(tile + unit_tile_bytes<D>());        // [keep_pad] byte offsets of the rows

    const char *Kh = reinterpret_cast<const char *>(K), *Vh = reinterpret_cast<const char *>(V);
    for (int t = lane; t < keep_pad; t += kWave) sl[t] = (unsigned)key(min(t, keep - 1)) * (D * 2u);

    // the sign of the scale goes into the query rows, its size into the exponential
    const float factor = fabsf(scale) * 1.44269504088896340736f;
    bf16x8 qop[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        uint4 raw = make_uint4(0, 0, 0, 0);
        if (c < vec) raw = *reinterpret_cast<const uint4 *>(Q + c * D + 32 * s + 8 * g);
        if (scale < 0.f) raw = Piece<uint16_t>::negate(raw);
        qop[s] = __builtin_bit_cast(bf16x8, raw);
    }
    wave_lds_sync();

    // gathers: lane (r = lane / LPR, p = lane % LPR) takes piece p of list entries VP r .. VP r + VP - 1 of the step, which
    // are also the tile's rows: the entries come as one or two 16-byte reads
    const int first = lane / LPR * VP;
    const unsigned piece = lane % LPR;
    v4u kring[DIRECT ? 1 : VP], vring[DIRECT ? 1 : VP];
    auto gather = [&](auto &ring, const char *head, int t0) {
#pragma unroll
        for (int r = 0; r < VP; r += 4) {
            const v4u at = *reinterpret_cast<const v4u *>(sl + t0 + first + r);
#pragma unroll
            for (int i = 0; i < 4; ++i) ring[r + i] = *reinterpret_cast<const v4u *>(head + (at[i] + 16u * piece));
        }
    };
    auto put = [&](const auto &ring) {
#pragma unroll
        for (int r = 0; r < VP; ++r)
            *reinterpret_cast<v4u *>(tile + (first + r) * ROW + 16u * (piece ^ unit_swizzle<D>(first + r))) = ring[r];
    };
    // DIRECT: request r fills the tile's rows RPI r .. RPI r + RPI - 1 with list entries in order, lane after lane 16 bytes, so that the lane of
    // place p in a row asks for piece p ^ unit_swizzle of the row (D = 128: another one in even and in odd requests)
    const unsigned group = lane / LPR, swizzled[2] = {16u * ((lane % LPR) ^ unit_swizzle<D>(group)), 16u * ((lane % LPR) ^ unit_swizzle<D>(RPI + group))};
    const unsigned base = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(__attribute__((address_space(3))) char *)tile);
    unsigned off[DIRECT ? VP : 1];
    auto find = [&](int t0) {
#pragma unroll
        for (int r = 0; r < VP; ++r) off[r] = sl[t0 + RPI * r + group] + swizzled[r & 1];
    };
    auto fetch = [&](const char *head) {
#pragma unroll
        for (int r = 0; r < VP; ++r)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(head + off[r]),
                                             (__attribute__((address_space(3))) void *)(size_t)(base + 1024u * r), 16, 0, 0);
    };
    // what was requested is in LDS; what was read from there is in registers, and may be overwritten
    auto fetched = [] { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };
    auto taken = [] { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); };
    // operands: row c (and 16 + c) of the key rows; of the value rows, the 4 x 4 block that ds_read_tr16_b64 takes from a lane
    const unsigned vrow = 4 * g + (c >> 2), vswz = unit_swizzle<D>(vrow);       // the same for row 16 + vrow
    auto key_piece = [&](int half, int s) {
        return *reinterpret_cast<const bf16x8 *>(tile + (16 * half + c) * ROW + 16u * ((4 * s + g) ^ unit_swizzle<D>(c)));
    };
    auto value_block = [&](int half, int ct) {
        return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (lds_s16x4 *)(tile + (16 * half + vrow) * ROW + 16u * ((2 * ct + (c >> 1 & 1)) ^ vswz) + 8 * (c & 1)));
    };

    v4f o[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) o[ct] = v4f{0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, z = 0.f;
    const float share = 1.f / (float)(keep_pad - keep + 1);      // the list is filled up with copies of its last key
    if constexpr (DIRECT) {
        find(0);
        fetch(Kh);
    } else {
        gather(kring, Kh, 0);
        gather(vring, Vh, 0);
    }
    for (int t0 = 0; t0 < keep_pad; t0 += 32) {
        const int t1 = min(t0 + 32, keep_pad - 32);
        bf16x8 keys[2][DIRECT ? KS : 1];
        if constexpr (DIRECT) {
            fetched();
#pragma unroll
            for (int half = 0; half < 2; ++half)
#pragma unroll
                for (int s = 0; s < KS; ++s) keys[half][s] = key_piece(half, s);
            taken();
            fetch(Vh);
            find(t1);
            __builtin_amdgcn_sched_barrier(0);
        } else {
            put(kring);
            gather(kring, Kh, t1);
            wave_lds_sync();
        }
        v4f s2[2];
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            s2[half] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                bf16x8 key;
                if constexpr (DIRECT) key = keys[half][s];
                else key = key_piece(half, s);
                s2[half] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(key, qop[s], s2[half], 0, 0, 0);
            }
        }
        if constexpr (!DIRECT) {
            wave_lds_sync();
            put(vring);
            gather(vring, Vh, t1);
        }
        float mx = fmaxf(s2[0][0], s2[1][0]);
#pragma unroll
        for (int i = 1; i < 4; ++i) mx = fmaxf(fmaxf(s2[0][i], s2[1][i]), mx);
        // (compared with >: nothing moves for scores that are not numbers, they reach the sums by themselves)
        if (__ballot(m == -INFINITY ? mx > -INFINITY : (mx - m) * factor > slack) != 0) {
            mx = fmaxf(mx, __shfl_xor(mx, 16, kWave));       // (through LDS: without it 1 to 3 % slower, N = 120, L = 1000, keep = 50, VEC = 4 66.9 and 68.7 us)
            mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));
            const float to = fmaxf(m, mx);
            const float f = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m - to) * factor);
            m = to;
            z *= f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float fi = __shfl(f, 4 * g + i, kWave);          // lane (query, 0): the sums of query 4 g + i
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) o[ct][i] *= fi;
            }
        }
        const float m0 = m == -INFINITY ? 0.f : m;
        float p[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) p[i] = __builtin_amdgcn_exp2f((s2[i / 4][i % 4] - m0) * factor);
        if (t0 + 32 > keep) {              // the copies of the last key share its weight: 0 would make NaN of an infinite value
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (t0 + 16 * (i / 4) + 4 * g + i % 4 >= keep - 1) p[i] *= share;
        }
        // A weight is the sum of two bf16 (relative 2^-16): one alone would be rounded at 2^-8, the largest one too, whose
        // weight is not 1 here.  hi is p cut off, and lo is not zero where p is not (the factor is 1 + 2^-23), so that both
        // products with an infinite value have its sign.
        unsigned cut[8];
        bf16x8 lo;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            z += p[i];
            cut[i] = __float_as_uint(p[i]) & 0xffff0000u;
            lo[i] = (__bf16)fmaf(p[i], 1.00000012f, -__uint_as_float(cut[i]));
        }
        const bf16x8 hi = __builtin_bit_cast(bf16x8, v4u{cut[0] >> 16 | cut[1], cut[2] >> 16 | cut[3], cut[4] >> 16 | cut[5], cut[6] >> 16 | cut[7]});
        union ValueBlock { s16x4 half[2]; bf16x8 all; };
        if constexpr (DIRECT) {
            fetched();
            ValueBlock vb[CT];
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                vb[ct].half[0] = value_block(0, ct);
                vb[ct].half[1] = value_block(1, ct);
            }
            taken();
            if (t0 + 32 < keep_pad) fetch(Kh);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                o[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi, vb[ct].all, o[ct], 0, 0, 0);
                o[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lo, vb[ct].all, o[ct], 0, 0, 0);
            }
        } else {
            wave_lds_sync();
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                ValueBlock vb;
                vb.half[0] = value_block(0, ct);
                vb.half[1] = value_block(1, ct);
                o[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi, vb.all, o[ct], 0, 0, 0);
                o[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lo, vb.all, o[ct], 0, 0, 0);
            }
            wave_lds_sync();                  // the next step overwrites the tile
        }
    }
    z += __shfl_xor(z, 16, kWave);
    z += __shfl_xor(z, 32, kWave);
    // lane (c, g) holds O[query 4g+i][16 ct + c]; the sum of query q sits in the lanes with column q
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float inv = 1.f / __shfl(z, 4 * g + i, kWave);
        if (4 * g + i < vec) {
            float *out = O + (4 * g + i) * D + c;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) out[16 * ct] = o[ct][i] * inv;
        }
    }
    float odd = 0.f;                       // NaN if a sum is not finite
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) odd = fmaf(o[ct][i], 0.f, odd);
    return __ballot(odd != 0.f) == 0;
}

// Weights above 1 may take large values beyond fp32 (from 2^111 / keep on) that weights of at most 1 would not: then once
// more with a reference that is the maximum.  (That from the start costs up to 13 % of the kernel.)
template <int D, bool DIRECT, typename Key>
__device__ __forceinline__ void attend_unit(const uint16_t *Q, const uint16_t *K, const uint16_t *V, Key &&key, float *O, int vec,
                                            int keep, int keep_pad, float scale, char *tile)
{
    for (float slack = kUnitSlack;; slack = 0.f) {
        int lane = threadIdx.x & (kWave - 1);
        asm volatile("" : "+v"(lane));     // nothing of a round is computed ahead of the loop: that would delay the first gathers
        if (unit_rows<D, DIRECT>(Q, K, V, key, O, vec, keep, keep_pad, scale, lane, tile, slack) || slack == 0.f) break;
    }
}

}  // namespace
}  // namespace dsa
