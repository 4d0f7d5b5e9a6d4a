// Exact attention of 16 neighbouring query rows (d = 64) with a list of kept keys each (paper section 3.4), by one workgroup on the bf16
// matrix cores, over the union of the lists.  What attention_tiles_bf16 and the predictor that goes on to attend share.
// Device code only; everything is internal to the translation unit that includes it.
#pragma once

#include "split_plan.h"
#include "unit_attend.h"

#include <algorithm>

namespace dsa {
namespace {

constexpr int kTileRows = 16;

// LDS of a workgroup of W wavefronts, in bytes from the start (every part a multiple of 16), with unions of up to `most` keys (a
// multiple of 32, at least 32).
struct TileLds {
    unsigned list, stats, work, bytes;
    __host__ __device__ TileLds(int W, int most)
    {
        list = 128;                                             // first: two words per wavefront; [most] entries of the union
        stats = list + most * 4;                                // [2][W][16]: references and sums of the wavefronts
        work = stats + 2 * W * kTileRows * 4;                   // a tile of 32 rows per wavefront, then its sums
        bytes = work + W * unit_tile_bytes<64>();
    }
};

// Whether `here` holds in any lane of the workgroup.  flags: a word per wavefront that nobody else uses until the next barrier.
__device__ __forceinline__ bool block_any(bool here, int *flags)
{
    const int wv = threadIdx.x / kWave, W = blockDim.x / kWave;
    const int any = __ballot(here) != 0;
    if (threadIdx.x % kWave == 0) flags[wv] = any;
    __syncthreads();
    int all = 0;
    for (int w = 0; w < W; ++w) all |= flags[w];
    return __builtin_amdgcn_readfirstlane(all) != 0;
}

__device__ __forceinline__ float max3(float a, float b, float c)
{
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// Entries behind the n of the union, up to a multiple of 32, that no row keeps: by one wavefront.
__device__ __forceinline__ void tile_fill(unsigned *entries, int n, int lane)
{
    if (n + lane < (n + 31) / 32 * 32) entries[n + lane] = 0;
}

// Dense lists overlap: 16 rows of 4096 keys that keep a tenth each have 3000 keys between them, not 6560.  Their key and value rows are
// gathered once for all 16, which is what a matrix instruction has columns for; a score that its row does not keep becomes -infinity, its
// weight 0.  The wavefronts take the steps of 32 keys in turn, each with sums and a running reference of its own (as in unit_rows), which are
// added up at the end.
// A weight of 0 does not keep an infinite or missing value out of a sum, and a reference that lags may take sums out of fp32: rows whose sums
// are not finite are done again one by one (attend_listed), with what they alone keep.  That is both routes' work: N = 16, L = 4096, keep = 410 with
// a value row of every head that is no number 420 us in one launch (row by row 298) instead of 240; given lists with a key twice are only
// told apart first, 244 by itself (224) instead of 157.
// A row's sums are of its own keys, but in the order of the union: their last bits depend on what the other rows of the tile keep, and on the
// plan's number of wavefronts.
// What bounds it: LDS, 8 writes of 14.3 cycles, 4 reads of 4.7 and 8 of 2.8 per step and CU (85 % of the time between the union and the sums),
// next to it vector issue (about 80 instructions per step; 73 %).  N = 16, L = 4096, keep = 410 in one launch with the predictor 301 -> 251
// us (row by row: 3.4 GB of gathers at 5 %, 6.9 GB at 10 %, now 3.1), 25 % 780 -> 387, by itself 224 -> 163 and 681 -> 285.  Tried: 32 rows per
// tile (81 steps instead of 118, but registers for one gather in flight: 117 -> 146 us), rows to LDS without registers (8 KB per wavefront
// instead of 4), the union from LDS atomics in the predictor (22 us instead of 8).
// nu rows (Q and O from the first of them on, K and V from the head on) over the n > 0 entries `key << 16 | rows that keep it` at
// lds + TileLds::list, filled up to a multiple of 32 (tile_fill) and seen by the whole workgroup.  Returns whether every sum was finite,
// the same in every wavefront.
__device__ __forceinline__ bool attend_tile(const uint16_t *Q, const uint16_t *K, const uint16_t *V, float *O, int nu, int n, float scale,
                                            int most, char *lds)
{
    constexpr int D = 64, ROW = D * 2, KS = D / 32, CT = D / 16, LPR = D / 8, VP = 32 * LPR / kWave;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = __builtin_amdgcn_readfirstlane(tid / kWave), T = blockDim.x, W = T / kWave;
    const int c = lane & 15, g = lane >> 4;
    const TileLds at(W, most);
    const unsigned *entries = reinterpret_cast<const unsigned *>(lds + at.list);
    float *s_m = reinterpret_cast<float *>(lds + at.stats), *s_z = s_m + W * kTileRows;
    char *tile = lds + at.work + wv * unit_tile_bytes<D>();
    const int pad = (n + 31) / 32 * 32;

    // the sign of the scale goes into the query rows, its size into the exponential
    bf16x8 qop[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        uint4 raw = make_uint4(0, 0, 0, 0);
        if (c < nu) raw = *reinterpret_cast<const uint4 *>(Q + c * D + 32 * s + 8 * g);
        if (scale < 0.f) raw = Piece<uint16_t>::negate(raw);
        qop[s] = __builtin_bit_cast(bf16x8, raw);
    }

    // ---- steps of 32 entries, a wavefront takes every W-th ----
    const float factor = fabsf(scale) * 1.44269504088896340736f;
    const char *Kh = reinterpret_cast<const char *>(K), *Vh = reinterpret_cast<const char *>(V);
    const int first = lane / LPR * VP;
    const unsigned piece = lane % LPR;
    v4u kring[VP], vring[VP];
    unsigned off[VP];
    auto find = [&](int t0) {
#pragma unroll
        for (int r = 0; r < VP; r += 4) {
            const v4u e = *reinterpret_cast<const v4u *>(entries + t0 + first + r);
#pragma unroll
            for (int i = 0; i < 4; ++i) asm("v_mad_u32_u16 %0, %1, %2, %3 op_sel:[1,0,0,0]" : "=v"(off[r + i]) : "v"(e[i]), "s"(ROW), "v"(16u * piece));      // (e >> 16) * ROW + ..
        }
    };
    auto gather = [&](v4u (&ring)[VP], const char *head) {
#pragma unroll
        for (int r = 0; r < VP; ++r) ring[r] = *reinterpret_cast<const v4u *>(head + off[r]);
    };
    auto put = [&](const v4u (&ring)[VP]) {
#pragma unroll
        for (int r = 0; r < VP; ++r) *reinterpret_cast<v4u *>(tile + (first + r) * ROW + 16u * (piece ^ unit_swizzle<D>(first + r))) = ring[r];
    };
    const unsigned vrow = 4 * g + (c >> 2), vswz = unit_swizzle<D>(vrow);       // the same for row 16 + vrow
    auto key_piece = [&](int half, int s) {
        return *reinterpret_cast<const bf16x8 *>(tile + (16 * half + c) * ROW + 16u * ((4 * s + g) ^ unit_swizzle<D>(c)));
    };
    auto value_block = [&](int half, int ct) {
        return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (lds_s16x4 *)(tile + (16 * half + vrow) * ROW + 16u * ((2 * ct + (c >> 1 & 1)) ^ vswz) + 8 * (c & 1)));
    };

    v4f o[CT], zs = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) o[ct] = v4f{0.f, 0.f, 0.f, 0.f};
    // row c's reference (of factor * score; exactly what the exponents are relative to), what is added to them, and the score that moves it
    float ref = -INFINITY, bias = 0.f, bound = -INFINITY;
    const float slack = kUnitSlack / factor;
    // (-1, 0) and (0, -1) in bf16, from registers: as constants of the instruction they would not mean the same in both halves
    unsigned minus[2] = {0x0000bf80u, 0xbf800000u};
    asm("" : "+s"(minus[0]), "+s"(minus[1]));
    bf16x8 ones;
#pragma unroll
    for (int i = 0; i < 8; ++i) ones[i] = (__bf16)1.f;
    int t0 = 32 * wv;
    if (t0 < pad) {
        // (in this order: the first round of the loop then waits for the keys only, as the others do)
        find(t0);
        gather(kring, Kh);
        __builtin_amdgcn_sched_barrier(0);
        gather(vring, Vh);
        __builtin_amdgcn_sched_barrier(0);
    }
    for (; t0 < pad; t0 += 32 * W) {
        put(kring);
        find(min(t0 + 32 * W, pad - 32));
        gather(kring, Kh);
        wave_lds_sync();
        v4f s2[2];
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            s2[half] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                s2[half] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(key_piece(half, s), qop[s], s2[half], 0, 0, 0);
            }
        }
        wave_lds_sync();
        put(vring);
        gather(vring, Vh);
        float s[8];
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const v4u e = *reinterpret_cast<const v4u *>(entries + t0 + 16 * half + 4 * g);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const unsigned kept = (unsigned)__builtin_amdgcn_sbfe((int)e[i], c, 1);
                s[4 * half + i] = __uint_as_float((__float_as_uint(s2[half][i]) & kept) | (0xff800000u & ~kept));
            }
        }
        const float mx = max3(max3(s[0], s[1], s[2]), max3(s[3], s[4], s[5]), max3(s[6], s[7], s[7]));
        if (__ballot(mx > bound) != 0) {
            const float top = halves_max<32>(halves_max<16>(mx));
            const bool moves = top > bound;
            const float to = moves ? top * factor : ref;
            const float f = !moves ? 1.f : ref == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ref - to);
            ref = to;
            bias = to == -INFINITY ? 0.f : -to;
            bound = moves ? top + slack : bound;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float fi = __shfl(f, 4 * g + i, kWave);          // lane (query, 0): the sums of query 4 g + i
                zs[i] *= fi;
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) o[ct][i] *= fi;
            }
        }
        float p[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) p[i] = __builtin_amdgcn_exp2f(fmaf(s[i], factor, bias));
        // a weight is the sum of two bf16 (relative 2^-17): one alone would be rounded at 2^-9, the largest one too, whose weight is not 1 here
        unsigned hi2[4], lo2[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            hi2[i] = __builtin_bit_cast(unsigned, bf16x2{(__bf16)p[2 * i], (__bf16)p[2 * i + 1]});
            const float a = Piece<uint16_t>::dot2(hi2[i], minus[0], p[2 * i]), b = Piece<uint16_t>::dot2(hi2[i], minus[1], p[2 * i + 1]);      // p - hi
            lo2[i] = __builtin_bit_cast(unsigned, bf16x2{(__bf16)a, (__bf16)b});
        }
        const bf16x8 hi = __builtin_bit_cast(bf16x8, v4u{hi2[0], hi2[1], hi2[2], hi2[3]}), lo = __builtin_bit_cast(bf16x8, v4u{lo2[0], lo2[1], lo2[2], lo2[3]});
        wave_lds_sync();
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            union { s16x4 half[2]; bf16x8 all; } vb;
            vb.half[0] = value_block(0, ct);
            vb.half[1] = value_block(1, ct);
            o[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi, vb.all, o[ct], 0, 0, 0);
            o[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lo, vb.all, o[ct], 0, 0, 0);
        }
        zs = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi, ones, zs, 0, 0, 0);
        zs = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lo, ones, zs, 0, 0, 0);
        wave_lds_sync();                  // the next step overwrites the tile
    }

    // ---- the wavefronts' shares, each with its own reference: lane (c, g) holds O[4g+i][16 ct + c] ----
    if (g == 0) s_m[wv * kTileRows + c] = ref;
    __syncthreads();
    // [16][D], where the wavefront's tile was, 16 columns at a time at those of another four for every four rows: on other banks
    float *part = reinterpret_cast<float *>(tile);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int q = 4 * g + i;
        const float mq = s_m[wv * kTileRows + q];
        float top = mq;
        for (int w = 0; w < W; ++w) top = fmaxf(top, s_m[w * kTileRows + q]);
        const float f = mq == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mq - top);
        if (c == 0) s_z[wv * kTileRows + q] = zs[i] * f;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) part[q * D + (16 * (ct ^ g) + c)] = o[ct][i] * f;
    }
    __syncthreads();
    float odd = 0.f;
    for (int e = 4 * tid; e < nu * D; e += 4 * T) {
        const int q = e / D;
        float z = 0.f;
        v4f sum = v4f{0.f, 0.f, 0.f, 0.f};
        for (int w = 0; w < W; ++w) {
            z += s_z[w * kTileRows + q];
            sum += *reinterpret_cast<const v4f *>(lds + at.work + w * unit_tile_bytes<D>() + (e ^ 16 * (q / 4)) * 4);
        }
        const float inv = 1.f / z;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            sum[i] *= inv;
            odd = fmaf(sum[i], 0.f, odd);
        }
        *reinterpret_cast<v4f *>(O + e) = sum;
    }
    return !block_any(odd != 0.f, reinterpret_cast<int *>(lds));
}

// The same rows by the loops of row_attend.h, from their lists in memory (entries clamped into [0, L), so that no list can send a gather
// outside K or V), which go through LDS, as many at a time as a.lds bytes have room for.
__device__ __forceinline__ void attend_listed(const AttendArgs &a, const int32_t *lists, char *lds, int L, int keep, unsigned n, int u0, int nu)
{
    uint16_t *image = reinterpret_cast<uint16_t *>(lds);
    const unsigned each = attend_rows_at_once<uint16_t>() * a.pad * sizeof(unsigned);                    // of a wavefront
    const int rows = min((int)((a.lds - each - 15) / (2 * keep)), nu);
    const unsigned room = (rows * keep * 2 + 15) / 16 * 16;
    for (int r0 = 0; r0 < nu; r0 += rows) {
        const int now = min(rows, nu - r0);
        __syncthreads();
        for (int e = threadIdx.x; e < now * keep; e += blockDim.x) image[e] = (uint16_t)min(max(lists[r0 * keep + e], 0), L - 1);
        __syncthreads();
        attend_block<uint16_t, 64>(a, image, reinterpret_cast<unsigned *>(lds + room), L, keep, 1, n, u0 + r0, now, (a.lds - room) / each);
    }
}

// ---- host side ----

// LDS of a workgroup: what attend_tile needs, and attend_listed for a row and a wavefront.
inline size_t tile_lds_bytes(const dsa_shape &sh, int W, int most)
{
    const size_t pad = (sh.keep + kRowPad - 1) / kRowPad * kRowPad;
    return std::max((size_t)TileLds(W, most).bytes, (size_t)sh.keep * 2 + 32 + attend_rows_at_once<uint16_t>() * pad * sizeof(unsigned));
}

// The longest union that rows of this shape can have, if they are attended over by attend_tile with W wavefronts per tile, else 0.
// A step of attend_tile serves 16 rows with 32 keys, whoever keeps them, a gather of attend_rows one row with 8.  Of 16 rows with a twelfth
// of the keys each, half to three quarters of all keys are in the union.  Lists that are given and lists that were just made have to take the
// same route; a line lies where neither is slower, or where one launch wins at least twice the microseconds that given lists lose.  Times of
// attend_rows and of attend_tile, k = 32 unless said, as one launch with the predictor and, in brackets, by itself; "random" are random codes,
// the others the low-rank inputs of the benchmark:
//   L >= 2048       5 %: N = 16, L = 4096 195 and 195 us (118 and 111), L = 2048 60 and 61 (31 and 35); a twelfth, random: N = 16, L = 2048 79.3
//                   and 75.9 (52.1 and 49.7), L = 4096 263 and 243 (189 and 161), N = 4, L = 8000 275 and 264 (181 and 159), N = 2, L = 11000
//                   326 and 265 (182 and 145), L = 16384 739 and 661 (488 and 404); 10 %: N = 16, L = 4096 301 and 251 (224 and 163), N = 64,
//                   L = 2048 323 and 275 (231 and 171); 25 %: 780 and 387 (681 and 285).
//   1024 to 2047    8.4 %, random: N = 64, L = 1024 94.0 and 93.2 (55.8 and 57.1), N = 20, L = 1500 65.6 and 64.3 (36.2 and 38.2), N = 32,
//                   L = 1030 64.1 and 64.8 (28.3 and 33.4); a ninth: L = 1030 79.8 and 70.7 (38.7 and 37.5), L = 1500 76.9 and 69.7.
//   640 to 1023     a ninth: N = 40, L = 700 45.8 and 44.6 (22.8 and 23.9), N = 100, L = 768 114 and 107 (66.0 and 61.7).
//   257 to 639      a sixth: N = 200, L = 300 69.2 and 63.4 (35.6 and 36.7), N = 60, L = 300 28.7 and 27.5 (12.6 and 15.2), N = 64, L = 512
//                   44.8 and 38.8 (27.1 and 24.0).
//   129 to 256      the fixed work of a row counts, not the gathers: two wavefronts per tile 13 to 40 % faster in one launch at any density
//                   (N = 192, L = 160, 2 keys 29.6 and 21.8 (11.5 and 8.1), L = 256, 26 keys 44.5 and 37.5; with 2048 to 2700 wavefronts up to 7 %
//                   slower by itself, N = 86, L = 177, 16 keys 20.3 and 15.6 (7.7 and 8.3)), four (few tiles) 4 to 7 % slower up to 10 %.
//   up to 128       10 %: N = 192, L = 128 24.0 and 25.0 (83 % of the speed by itself).
//   a round of      (little of a second one, which attend_rows spreads over the chip row by row) an eighth: N = 27, L = 640 37.9 and 35.7 (15.2
//   4096 wavefronts and 17.8), N = 22, L = 768 39.0 and 36.4 (17.5 and 19.7), N = 21, L = 800 41.2 and 37.0 (18.1 and 19.5); a seventh: N = 26,
//   and up to half  L = 640 39.4 and 36.1 (17.1 and 18.5); a ninth: N = 17, L = 1024 40.7 and 36.6 (20.6 and 22.1); a twelfth: N = 9, L = 2048
//   a round         55.9 and 50.6 (28.8 and 29.5), N = 1, L = 8200 121 and 109 (56.1 and 60.0), N = 2, L = 5200 85.1 and 78.7 (41.7 and 43.4).
//   less than one   a ninth: N = 8, L = 1024 22.2 and 22.1 (11.3 and 13.1), 10 %: N = 4, L = 2048 31.7 and 30.4 (17.0 and 19.1); a fifth: 28.8
//                   and 23.8, 46.4 and 35.4, N = 13, L = 640 28.0 and 24.2 (12.6 and 12.9); a quarter N = 31, L = 257 20.5 and 16.6 (9.2 and 9.9).
//                   Eight wavefronts per tile of a short head (up to 1024): a fifth N = 7, L = 640 19.0 and 19.1 (8.5 and 10.5), N = 5, L = 900
//                   23.4 and 22.2 (10.7 and 12.2), L = 1000 24.9 and 22.5 (11.9 and 13.0); a quarter N = 7, L = 640 21.2 and 19.3 (10.0 and 11.1),
//                   N = 6, L = 768 23.2 and 20.5 (11.3 and 11.7); a third N = 7, L = 640 0.81 of the time (0.92).
//   one workgroup   unions whose list and tiles take more than 80 KB (L > 12032) leave a CU eight wavefronts instead of sixteen: a twelfth
//   per CU          N = 1, L = 12600 262 and 278 (147 and 159), N = 2, L = 13000 489 and 506 (274 and 285), N = 4, L = 14500 1260 and 1290
//                   (742 and 761), L = 15500 1532 and 1435 (966 and 867); a tenth 1008 and 1013 (637 and 619) with N = 4, L = 12600, N = 2,
//                   L = 13000 606 and 559 (375 and 320).
//   rounds of      (two wavefronts in turn for every place, and codes of low rank, rank 32, with and without high-norm keys: the unions of uniformly
//   4096 waves     random codes are longer, and lose 1 to 5 % at 5 %, 0 to 4 % at a sixteenth) 5 %: N = 16, L = 4096 187 to 192 and 179 to 185 (118 and
//                  114), INT4, both passes of the projection included, 242 and 230, N = 12 140 to 146 and 139 to 147 (92 and 88), N = 32 375 and 361
//                  (238 and 228), N = 20, L = 3600 208 to 215 and 203 to 205 (117 and 115), N = 16, L = 5000 290 and 275 (181 and 164); a sixteenth: N = 8,
//                  L = 4096 112 and 106 to 112 (73 and 71), N = 8, L = 5000 181 and 175 (109 and 101), N = 40, L = 3000 318 and 300 (199 and 181), N = 64,
//                  L = 2048 242 and 226 (150 and 146), N = 20 81 to 87 and 81 to 83 (49 and 51; 7 % 87 and 83, 57 and 53); 5 %, N = 8, L = 4096 99.6 and 101 (58.8 and
//                  62.2), N = 40, L = 3000 274 and 274 (156 and 161), N = 8, L = 8000 365 and 386 (211 and 213), 6 %, N = 12, L = 6000 340 and 361; a thirteenth: N = 128,
//                  L = 1024 173 and 164 (102 and 100), N = 100, L = 1500 262 and 244 (163 and 145), but N = 40, L = 1024 62.2 and 62.4 (33.5 and 34.7); a
//                  tenth: N = 80, L = 700 82.8 and 77.8 (43.3 and 42.5), N = 100, L = 900 139 and 128 (80 and 75); an eighth: N = 96, L = 512 48.2 and 49.4
//                  (32.4 and 33.0).
//   the line at    codes of low rank cross at 4 to 5 %, uniformly random ones at 5.5 to 6 %, and it lies between.  In one launch, low rank and random:
//   5 %            N = 16, L = 4096 4 % 184/184 and 183/191, 4.5 % 188/180 and 181/192, 5 % 192/186 and 193/199, 5.5 % 212/196 and 210/211; N = 32 4 % 348/337 and 348/360,
//                  5 % 390/375 and 386/388; N = 12 4 % 135/134 and 130/139, 5 % 153/147 and 147/152; N = 16, L = 3600 4.5 % 168/166 and 167/175, 5 % 172/171 and 173/181, 5.5 %
//                  183/179 and 182/186; N = 20, L = 4500 4.5 % 285/286 and 288/298, 5 % 309/299 and 312/318; N = 16, L = 5000 4 % 265/260 and 257/271, 5 % 291/281 and 292/300.
//                  (Norms that vary and clusters make unions shorter: N = 16, L = 4096, 5 %, log-normal norms 204/170, 5 % of the keys with four times the norm 190/175, eight
//                  clusters 203/196.)
// Wider rows of K and V (d = 128) do not leave the registers, fp32 has no matrix instruction of that rate.
// A scale of 0 makes 0 * -infinity, no number, of the exponent of a key that a row does not keep: every tile would be done again row by row
// (N = 16, L = 4096, keep = 410 299 and 431 us, by itself 224 and 349).
inline int tile_most(const dsa_shape &sh, int W)
{
    if (W < 1 || W > 8 || 2 * sh.L > W * unit_tile_bytes<64>()) return 0;
    const long long waves = (long long)sh.B * sh.H * ((sh.L + kTileRows - 1) / kTileRows) * W;
    const int part = tile_part(sh, waves);
    if (!part) return 0;
    const int most = (std::min((long long)sh.L, (long long)kTileRows * sh.keep) + 31) / 32 * 32;
    const size_t lds = tile_lds_bytes(sh, W, most);
    if (lds > 128 * 1024) return 0;
    if (sh.L <= 256) return W == 2 ? most : 0;
    int share = part;
    if (waves < 4096) share = std::min(share, W < 8 || sh.L > 1024 ? 5 : sh.L < 768 ? 3 : sh.L < 960 ? 4 : 5);
    else if (waves > 4096 && waves < 6144 && sh.L < 800) share = std::min(share, 7);
    if (lds > 80 * 1024 && sh.L < 15000) share = std::min(share, 10);
    return (long long)sh.keep * share >= sh.L ? most : 0;
}

}  // namespace
}  // namespace dsa
