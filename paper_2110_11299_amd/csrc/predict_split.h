// The mask predictor (paper section 3.1: approximate scores S~ = Q~ K~^T and the per-unit top-k that becomes the mask;
// section 5.1: a unit is a query row, or a group of 4 / 8 rows whose scores are summed).  Scores are exact integers, so
// the selection is exact: larger score first, lower key index among equals, list ascending.  No score is ever stored:
// the int8 contraction is cheap enough on the matrix cores to be swept twice.
//
// One workgroup of W wavefronts owns 16 * UT units of one head and the wavefronts split its keys.  Keys are the rows
// (A operand), units the columns (B operand) of v_mfma_i32_16x16x64_i8; the key range is cut into 4 W lane ranges of
// 32 * NW keys, and lane (c = lane % 16, g = lane / 16) of wavefront w holds, for unit c, the scores of range 4 w + g.
//
//   sweep 1    every lane keeps up to NB = 32 or 16 maxima over disjoint key sets ("buckets").
//   bounds     from a histogram of the upper part of a unit's maxima in LDS two thresholds tl < th are read off, such that the keep-th
//              largest score lies between them almost surely: the number of buckets that the x largest keys fall into
//              is known to a few per cent (section "targets" on the host side).  What lies outside of the part has a second
//              histogram.  For short ranges a bucket is one key.
//   sweep 2    the keys are swept again with -tl as accumulator input: the signs of what comes out and of that less th - tl are two
//              bitmaps (of NW words per lane; the band between them stays in registers, the other goes to LDS), and their counts.
//   check      count(>= th) <= keep <= count(>= tl), and few enough keys between (the "band"): else the bracket is
//              moved or cut in three and swept again.  This ends for any scores: the bracket shrinks until it holds a
//              single score value, and a plateau of equal scores needs no score at all (its first keys are taken).
//   band       only the keys between the thresholds (about 50 of 4096) get their scores recomputed, from K~ rows, 16
//              lanes per unit; the exact threshold is found by interpolation and bisection in turn, ties go to the lower key.
//   emission   every lane turns its words into key indices at its place in the unit's row, in LDS; the rows leave as
//              one contiguous block.
//   attention  where it pays, over the lists while they are in LDS (row_attend.h, unit_attend.h), or over their union, which comes from the
//              bitmaps in the registers (tile_attend.h).
//
// What bounds it: vector-ALU issue (half an operation per score in sweep 1, three of half the cycles in sweep 2, about 25 per candidate).
// Add, and, three-way logic and fma take two cycles per wavefront here, everything with a scalar operand, shifts to the left, compares, minima and
// most of what has three operands four.
// Splitting the keys rather than giving a wavefront whole units keeps the bitmaps in registers, needs a quarter of the
// bucket registers per lane and gives every shape, the shortest included, four times the wavefronts.
#pragma once

#include "dsa_internal.h"
#include "predict_api.h"
#include "split_bounds.h"
#include "split_plan.h"
#include "key_rows.h"
#include "key_stream.h"
#include "tile_attend.h"

#include <math.h>

#include <algorithm>

namespace dsa {
namespace {

constexpr int kBelow = 4;               // words before them, one for each lane of a unit in a wavefront: what lies below the bins, mostly, goes there without a conflict
constexpr int kBinStride = kBins + kBelow;      // words from unit to unit: the units' bins start in different banks
// Keys of one unit's band that are scored, 16 per slot.  Few-level codes make bands of whole plateaus of equal scores, which are swept
// again where they do not fit: INT4 codes at L = 4096, keep = 205, 16 high-norm keys per head, with 24 slots 146.7 us (unpacking
// included), with 32 138.4.  Where that does not pay (short ranges, whose bands are one bucket, and units of several rows, which
// have many levels) or the registers are short (two tiles), it is 24.
template <bool GROUP, int UT, int NWM> constexpr int band_slots() { return !GROUP && UT == 1 && NWM >= 4 ? 32 : 24; }
// Slots that are looked at together: their requests are on their way at the same time.  Of two instead of four, bands of more than 32 keys
// wait twice as often: N = 4, L = 1024, k = 32, keep = 204 and 341 12.6 and 14.1 us, 14.5 and 17.0; N = 16, L = 4096, keep = 205 190.9 and 195.6.
constexpr int kBandStep = 4;

// The attention that a workgroup goes on with, over the lists it has just made (see attend_here): fp32 rows, bf16 rows (of units
// of several rows: the units on the matrix cores), or bf16 rows over the union of their lists, on the matrix cores.
enum AttendKind { kNoAttend, kAttendF32, kAttendBf16, kAttendTile };

struct SplitArgs {
    const int8_t *Qt, *Kt;
    int32_t *idx;
    int L, k, keep, vec;
    int NW;                             // bitmap words per lane: a lane range is 32 * NW keys
    int wgs_per_head;
    int target_l, target_h;             // buckets that reach tl / th
    float low, high;                    // the histogram's window (SplitPlan)
    int direct;                         // the rows do not fit LDS: indices go straight to memory
};
struct SplitAttendArgs : SplitArgs { AttendArgs attend; };

// LDS of a workgroup, in bytes from the start (every part a multiple of 16).
struct SplitLds {
    unsigned tot, q, hist, list, bytes;
    unsigned sel;                                               // words from unit to unit of the bitmaps at `hist`, one more than they have: other banks
    unsigned attend;                                            // what the attention needs, behind the image of the rows
    __host__ __device__ SplitLds(int W, int UT, int NW, int k, bool group, int keep, bool direct, int slots)
    {
        const unsigned U = kTile * UT;
        tot = 6 * U * 4;                                        // [6][U]: tl, th, need (smallest maximum before), band count (flags before), base and shift of the bins
        q = tot + 2 * W * U * 4;                                // [2][W][U]
        hist = q + U * (group ? 2 : 1) * (k + 16);              // [U][parts][k + 16]
        sel = 4 * W * NW + 1;
        const unsigned h = U * kBinStride * 4, s = (U * sel * 4 + 15) / 16 * 16;
        list = hist + (h > s ? h : s);                          // [U][bins], later the bitmaps of kept keys [U][sel]
        bytes = list + U * slots * 16 * 2;                      // [U][16 slots]
        const unsigned rows = hist + (direct ? 0 : (U * keep * 2 + 16 + 15) / 16 * 16);   // image of the index rows, last
        if (rows > bytes) bytes = rows;
        attend = rows;
    }
};

// x from the lane whose number differs by `bit`.
template <int bit> __device__ __forceinline__ int dpp_xor(int x)
{
    if constexpr (bit == 1) return dpp_move<kDppXor1>(x);
    else if constexpr (bit == 2) return dpp_move<kDppXor2>(x);
    else return dpp_move<0x1B>(dpp_move<kDppHalfMirror>(x));         // 4: ^ 7, then ^ 3
}
// Words from the signs of 32 numbers below 2^24, whose upper eight bits are all alike: number i puts its sign at bit 24 + i % 8 of part i / 8, in this
// order but for 7 before 6.  The first fills the part, and the masks of the others reach over bits that the ones behind them take, so that
// four of them are constants of the instruction and four are in registers: v_bitop3 takes two cycles per wavefront (a funnel shift or v_bfi
// four), but not with a scalar operand.  Sweep 2 with it and with y = x - (th - tl) instead of a second matrix instruction (19 cycles for
// four scores, as long as all else): mask, N = 16, L = 2048, k = 64, keep = 102 46.6 -> 41.2 us, N = 4, L = 16384, k = 64 390 -> 371, N = 16, L = 4096, k = 32,
// keep = 205 94.6 -> 91.6.
struct SignMasks {
    unsigned reg[4];
    __device__ __forceinline__ SignMasks()
    {
        reg[0] = 0x3c000000u; reg[1] = 0x38000000u; reg[2] = 0x30000000u; reg[3] = 0x20000000u;
#pragma unroll
        for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(reg[i]));
    }
    __device__ __forceinline__ void put(unsigned &part, int i, int x) const
    {
        const unsigned mask = i == 1 ? 0x3e22f983u /* 1 / (2 pi) */ : i == 7 ? 0xc0000000u /* -2.0 */ : i == 6 ? 0x40000000u /* 2.0 */ : reg[(i - 2) & 3];
        part = i == 0 ? (unsigned)x : __builtin_amdgcn_bitop3_b32(mask, (unsigned)x, part, 0xCA);         // (mask & x) | (~mask & part)
    }
    // numbers first, first + 1, .. of the 32
    template <typename V> __device__ __forceinline__ void tile(unsigned (&part)[4], int first, const V &x) const
    {
        constexpr int N = sizeof(V) / sizeof(int);
#pragma unroll
        for (int r = 0; r < N; ++r) {
            const int i = (first + r) % 8, now = i == 6 ? r + 1 : i == 7 ? r - 1 : r;
            put(part[(first + now) / 8], (first + now) % 8, x[now]);
        }
    }
    static __device__ __forceinline__ unsigned word(const unsigned (&part)[4])
    {
        return __builtin_amdgcn_perm(part[1], part[0], 0x0c0c0703u) | __builtin_amdgcn_perm(part[3], part[2], 0x07030c0cu);
    }
};

// Sum / maximum over the 16 lanes of a row (DPP).
__device__ __forceinline__ int row_sum(int x)
{
    x += dpp_move<kDppXor1>(x);
    x += dpp_move<kDppXor2>(x);
    x += dpp_move<kDppHalfMirror>(x);
    return x + dpp_move<kDppMirror>(x);
}
__device__ __forceinline__ int row_max(int x)
{
    x = max(x, dpp_move<kDppXor1>(x));
    x = max(x, dpp_move<kDppXor2>(x));
    x = max(x, dpp_move<kDppHalfMirror>(x));
    return max(x, dpp_move<kDppMirror>(x));
}
// Sums of N values over N neighbouring lanes: lane l gets that of value l % N.
template <int N> __device__ __forceinline__ int key_sums(const int (&x)[N], int lane)
{
    if constexpr (N == 1) {
        return x[0];
    } else {
        constexpr int H = N / 2;
        int y[H];
#pragma unroll
        for (int i = 0; i < H; ++i) {
            const int lower = x[i] + dpp_xor<H>(x[i]), upper = x[i + H] + dpp_xor<H>(x[i + H]);
            y[i] = lane & H ? upper : lower;
        }
        return key_sums<H>(y, lane);
    }
}
// Sum of x over the lanes above this one in its row of 16.
__device__ __forceinline__ int row_sum_above(int x)
{
    int s = x;
    s += __builtin_amdgcn_update_dpp(0, s, 0x101, 0xF, 0xF, true);   // row_shl:1
    s += __builtin_amdgcn_update_dpp(0, s, 0x102, 0xF, 0xF, true);   // row_shl:2
    s += __builtin_amdgcn_update_dpp(0, s, 0x104, 0xF, 0xF, true);   // row_shl:4
    s += __builtin_amdgcn_update_dpp(0, s, 0x108, 0xF, 0xF, true);   // row_shl:8
    return s - x;
}

// The workgroup's nu units of vec rows, one at a time per wavefront.  lds: room for a tile and the list per wavefront.
template <int D>
__device__ __forceinline__ void attend_block_units(const AttendArgs &a, const uint16_t *image, char *lds, int L, int keep, int vec, unsigned n, int u0, int nu)
{
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), W = blockDim.x / kWave;
    const size_t head = (size_t)n * L * D;
    const uint16_t *Q = static_cast<const uint16_t *>(a.Q), *K = static_cast<const uint16_t *>(a.K) + head, *V = static_cast<const uint16_t *>(a.V) + head;
    for (int u = wv; u < nu; u += W) {
        const size_t first = head + (size_t)(u0 + u) * vec * D;
        attend_unit<D, false>(Q + first, K, V, [&](int t) { return (int)image[u * keep + t]; }, a.O + first, vec, keep, a.pad, a.scale,
                       lds + wv * (unit_tile_bytes<D>() + a.pad * 4));
        wave_lds_sync();                   // the next unit overwrites list and tile
    }
}

// Bits of a square of 16 x 16, twice: lane c of a row of 16 has row c in its lower half word (and another square's in the upper one) and
// gets column c.
struct Transpose16 {
    unsigned amount[4], stays[4];
    __device__ __forceinline__ explicit Transpose16(int c)
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const unsigned s = 1u << i, low = i == 0 ? 0x55555555u : i == 1 ? 0x33333333u : i == 2 ? 0x0f0f0f0fu : 0x00ff00ffu;
            amount[i] = c & s ? s : 32 - s;            // what comes from the other lane goes s down or up
            stays[i] = c & s ? ~low : low;
        }
    }
    __device__ __forceinline__ unsigned step(unsigned x, unsigned other, int i) const
    {
        return (x & stays[i]) | (__builtin_amdgcn_alignbit(other, other, amount[i]) & ~stays[i]);
    }
    __device__ __forceinline__ unsigned operator()(unsigned x) const
    {
        x = step(x, (unsigned)dpp_move<0x128>((int)x), 3);                                     // lane ^ 8 (row_ror:8)
        x = step(x, (unsigned)dpp_move<0x1B>(dpp_move<kDppHalfMirror>((int)x)), 2);            // lane ^ 4: ^ 7, then ^ 3
        x = step(x, (unsigned)dpp_move<kDppXor2>((int)x), 1);
        return step(x, (unsigned)dpp_move<kDppXor1>((int)x), 0);
    }
};

// The union of the lists of a tile's units from their bitmaps: word w of a lane holds the keys first + 32 w .. of unit c that are kept
// (live: the unit exists).  Entries as in tile_attend.h, keys ascending.  Returns their number.  counts: a word per wavefront.  What was at
// `entries` may be read until the barrier in here.
template <int NWM>
__device__ __forceinline__ int union_entries(const unsigned (&words)[NWM], int NW, int first, bool live, unsigned *entries, int *counts)
{
    const int lane = threadIdx.x & (kWave - 1), wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), W = blockDim.x / kWave;
    const int c = lane & 15, g = lane >> 4;
    const Transpose16 transpose(c);
    unsigned m[NWM];                       // keys first + 32 w + c and 16 more: the units that keep them, 16 bits each
    int mine = 0;
#pragma unroll
    for (int w = 0; w < NWM; ++w) {
        m[w] = 0;
        if (w < NW) {
            m[w] = transpose(live ? words[w] : 0u);
            mine += ((m[w] & 0xffffu) != 0) + ((m[w] >> 16) != 0);
        }
    }
    int all;
    int pos = unit_excl_scan(row_sum(mine), g, &all);
    if (lane == 0) counts[wv] = all;
    __syncthreads();
    int total = 0;
    for (int w = 0; w < W; ++w) {
        pos += w < wv ? counts[w] : 0;
        total += counts[w];
    }
    total = __builtin_amdgcn_readfirstlane(total);
    if (wv == 0) tile_fill(entries, total, lane);
    const unsigned below = (1u << c) - 1u, shift = 16 * (g & 1);
#pragma unroll
    for (int w = 0; w < NWM; ++w) {
        if (w < NW) {
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const bool kept = half ? m[w] >> 16 : m[w] & 0xffffu;
                const unsigned long long b = __ballot(kept);
                const unsigned row = ((g & 2 ? (unsigned)(b >> 32) : (unsigned)b) >> shift) & 0xffffu;      // of the keys that this row of lanes has
                const unsigned key = first + 32 * w + 16 * half + c;
                if (kept) entries[pos + __popc(row & below)] = half ? __builtin_amdgcn_alignbit(key, m[w], 16) : (key << 16) | (m[w] & 0xffffu);
                pos += __popc(row);
            }
        }
    }
    __syncthreads();
    return total;
}

// Wavefronts per SIMD.  Ranges of one group need few registers: rows by themselves and with bf16 attention fit 96 (up to 8 more through
// scratch at k = 48 and 64), of 115 that they would take.  Four and five: N = 96, L = 512, k = 32, keep = 25 22.8 and 21.6 us, with attention
// 42.1 and 39.4.  fp32 attention and tiles do not fit (a forward of N = 300, L = 256, keep = 25 46.6 and 53.5), groups of rows gain nothing.
template <int NWM, bool GROUP, int ATTEND> constexpr int split_waves_per_simd()
{
    return NWM == 1 && !GROUP && (ATTEND == kNoAttend || ATTEND == kAttendBf16) ? 5 : 4;
}

// K: the projection dimension (16, 32, 48, 64, 128), or 0 for any other (up to 112, two contraction steps).
// GROUP: units are groups of vec rows.  UT: tiles of 16 units per workgroup.  NB: buckets per lane and unit (32, or 16 if a
// range has several groups).  NWM: most bitmap words per lane.
// ATTEND: the attention that it goes on with, an instance of its own for each kind (the one without is up to 3 % faster for it; fp32
// rows and bf16 units in one instance kept 103 registers in scratch: groups of 8, k = 32, N = 32, L = 8192, keep = 82 198 us, now 146).
template <int K, bool GROUP, int UT, int NB, int NWM, int ATTEND>
__global__ __launch_bounds__(NWM >= 8 ? 1024 : 512, (split_waves_per_simd<NWM, GROUP, ATTEND>())) void predict_split(
    std::conditional_t<ATTEND != kNoAttend, SplitAttendArgs, SplitArgs> a)
{
    constexpr int R = K == 16 ? 4 : K == 32 ? 2 : 1;     // keys side by side in a matrix row = tiles per row operand
    constexpr int STEPS = K && K <= 64 ? 1 : 2;          // contraction steps of 64
    // Rows of 128 bytes: the four rows that neighbouring lanes read 16 bytes of lie at the same place of their cache lines, and
    // the L1 takes them one after the other.  Odd rows fetch their second half first, and the halves change places in front
    // of the matrix instruction.  L = 4096, keep = 41, N = 8: 251 -> 143 us (k = 112, whose rows spread by themselves: 111).
    constexpr bool CROSS = K == 128;
    // Rows of 64 bytes: two of the four rows that neighbouring lanes read 16 bytes of lie at the same place of their cache lines.  In
    // sweep 1, which waits for the L1, every other pair of rows is fetched with its halves exchanged and multiplied with the units'
    // halves exchanged: a second matrix instruction per tile, which leaves the right scores in the registers of those rows.  (In
    // sweep 2 vector and matrix instructions are the longer.)  N = 4, L = 16384: sweep 1 129 -> 84 us, a call 651 -> 615; N = 8, L = 8192,
    // keep = 82, groups of 8 57.3 -> 54.0.  Two tiles of groups have no registers for it: N = 16, L = 8192, d = 128 120 and 130 us.
    constexpr bool TWIST = K == 64 && !(GROUP && UT == 2);
    constexpr int NS = 8 / R;                            // row operands of a group of 8 tiles (32 keys per lane range)
    constexpr int NSB = key_batch_slots(NS, STEPS, GROUP && UT == 1 && K != 48);    // row operands of one batch of requests (8 registers each if two steps)
    constexpr int BPG = NS / NSB;                        // batches per group
    constexpr int TB = NSB * R;                          // tiles per batch
    constexpr int PAIR = TB >= 4 ? 2 : 1;                // tiles j and j + PAIR share a bucket
    constexpr int PARTS = GROUP ? 2 : 1;
    constexpr int U = kTile * UT;
    constexpr int kBandSlots = band_slots<GROUP, UT, NWM>(), kBandCap = 16 * kBandSlots;
    constexpr int SG = kBandStep;
    constexpr bool AGAIN = split_bins_again(K, GROUP, NWM);              // (K = 0 is no multiple of 16 up to 64)
    constexpr bool COPIES = !((K == 0 || K == 128) && GROUP);            // |score - threshold| < 2^24 (SignMasks)
    // Lanes that fetch a key row of the band, 16 bytes each: the L1 looks a row up once, not once for every 16 bytes.  N = 4, L = 16384, k = 64,
    // keep = 164 band scores and search 51 -> 29 us; N = 16, L = 4096, k = 32, keep = 205 96.8 -> 94.6 in all.  (k = 128: 100 to 800 registers through
    // scratch; single keys as buckets, k = 64: 49, and bands are a few keys.)
    constexpr int LPK = NWM > 1 && (K == 32 || K == 64) ? K / 16 : 1;
    extern __shared__ __align__(16) unsigned char lds[];

    const int k = K ? K : a.k;
    const int L = a.L, keep = a.keep, NW = a.NW, Lr = 32 * NW;
    const int T = blockDim.x, W = T / kWave;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int c = lane & 15, g = lane >> 4, h = 4 * wv + g;
    const SplitLds at(W, UT, NW, k, GROUP, keep, a.direct, kBandSlots);
    int *s_tl = reinterpret_cast<int *>(lds), *s_th = s_tl + U, *s_need = s_th + U, *s_nb = s_need + U, *s_base = s_nb + U, *s_shift = s_base + U;
    int *s_totl = reinterpret_cast<int *>(lds + at.tot), *s_toth = s_totl + W * U;       // [W][U] each
    unsigned char *s_q = lds + at.q;
    const int qstride = PARTS * (k + 16);
    unsigned *hist = reinterpret_cast<unsigned *>(lds + at.hist);
    uint16_t *list = reinterpret_cast<uint16_t *>(lds + at.list);

    const unsigned wg = xcd_contiguous(blockIdx.x, gridDim.x);
    const unsigned n = wg / (unsigned)a.wgs_per_head;
    const int u0 = (int)(wg % (unsigned)a.wgs_per_head) * U;
    const int G = GROUP ? L / a.vec : L;
    const int nu = min(U, G - u0);
    const int8_t *Kh = a.Kt + (size_t)n * L * k;
    const int8_t *Qh = a.Qt + (size_t)n * L * k;

    // ---- query side of every unit into LDS: the row, or the sum of the unit's rows as 128 hi + lo -----------------
    for (int e = tid; e < U * (k / 4); e += T) {
        const int u = e / (k / 4), c4 = e - u * (k / 4);
        int lo = 0, hi = 0;
        if (u < nu) {
            if (GROUP) {
                const int *row = reinterpret_cast<const int *>(Qh + (size_t)(u0 + u) * (a.vec * k)) + c4;
                int sum[4] = {0, 0, 0, 0};
                for (int r = 0; r < a.vec; ++r) add_bytes(sum, row[r * (k / 4)]);
                split_sums(sum, lo, hi);
            } else {
                lo = reinterpret_cast<const int *>(Qh + (size_t)(u0 + u) * k)[c4];
            }
        }
        int *dst = reinterpret_cast<int *>(s_q + u * qstride) + c4;
        dst[0] = lo;
        if (GROUP) dst[(k + 16) / 4] = hi;
    }
    for (int e = tid; e < U * kBinStride / 4; e += T) reinterpret_cast<v4i *>(hist)[e] = v4i{0, 0, 0, 0};

    // ---- key rows: lane (r = lane % 16, kb = lane / 16) fetches 16 bytes of matrix row r (key_rows.h) ---------------
    // (buffer loads: the batch is in the base and the length of the descriptor, scalar work, the row operand an immediate offset;
    // rows beyond L read zeros without a test)
    const int sub = R == 4 ? g : R == 2 ? g >> 1 : 0;
    unsigned poff[STEPS], voff[STEPS];
    bool plive[STEPS];
    const bool crossed = CROSS && (c & 1);
    const unsigned row0 = key_row_offset(wv, lane, Lr, k, R);
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
        plive[s] = key_piece_offset(lane, k, R, s) >= 0;
        poff[s] = max(key_piece_offset(lane, k, R, s), 0);
    }
#pragma unroll
    for (int s = 0; s < STEPS; ++s) voff[s] = row0 + poff[crossed ? STEPS - 1 - s : s];
    unsigned twisted[STEPS];
#pragma unroll
    for (int s = 0; s < STEPS; ++s) twisted[s] = TWIST && (c & 2) ? row0 + (poff[s] ^ 32u) : voff[s];
    const int slot_step = key_slot_step(k, R);
    int batches = NW * BPG;
    auto request = [&](v4i (&dst)[NSB][STEPS], int b, const unsigned (&at)[STEPS]) {          // batches beyond the range read its last one
        const int first = __builtin_amdgcn_readfirstlane(key_batch_offset(b, batches, NSB, slot_step));
#pragma unroll
        for (int sl = 0; sl < NSB; ++sl) {
            const int from = K ? first : first + sl * slot_step;
            const __amdgpu_buffer_rsrc_t keys =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t *>(Kh) + from, 0, key_bytes_left(L, k, from), 0x00020000);
#pragma unroll
            for (int s = 0; s < STEPS; ++s)
                dst[sl][s] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(keys, K ? at[s] + sl * slot_step : at[s], 0, 0));
        }
        __builtin_amdgcn_sched_barrier(0);       // the requests stay ahead of the batch that is used next
    };
    v4i rows[2][NSB][STEPS];
    request(rows[0], 0, twisted);
    __syncthreads();

    // unit operands: 16 bytes of the unit's query side where this lane's part of the key row is, zero in the tiles of
    // the row operand that belong to other keys
    v4i q[UT][PARTS][R][STEPS];
#pragma unroll
    for (int t = 0; t < UT; ++t)
#pragma unroll
        for (int p = 0; p < PARTS; ++p)
#pragma unroll
            for (int s = 0; s < STEPS; ++s) {
                const v4i piece = *reinterpret_cast<const v4i *>(s_q + (kTile * t + c) * qstride + p * (k + 16) + poff[s]);
#pragma unroll
                for (int i = 0; i < R; ++i) q[t][p][i][s] = (sub == i && plive[s]) ? piece : v4i{0, 0, 0, 0};
            }

    v4i qx[UT][PARTS];                                   // with the halves exchanged, for sweep 1
#pragma unroll
    for (int t = 0; t < UT; ++t)
#pragma unroll
        for (int p = 0; p < PARTS; ++p)
            if (TWIST) qx[t][p] = *reinterpret_cast<const v4i *>(s_q + (kTile * t + c) * qstride + p * (k + 16) + (poff[0] ^ 32u));

    // scores of tile j of the batch against the units of operand t, each plus b
    auto tile_scores = [&](const v4i (&buf)[NSB][STEPS], int j, int t, int b) -> v4i {
        v4i key[STEPS];
#pragma unroll
        for (int s = 0; s < STEPS; ++s)
#pragma unroll
            for (int i = 0; i < 4; ++i) key[s][i] = CROSS && crossed ? buf[j / R][STEPS - 1 - s][i] : buf[j / R][s][i];
        v4i acc = v4i{b, b, b, b};
#pragma unroll
        for (int s = 0; s < STEPS; ++s) acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(key[s], q[t][0][j % R][s], acc, 0, 0, 0);
        if (GROUP) {
            v4i top = v4i{0, 0, 0, 0};
#pragma unroll
            for (int s = 0; s < STEPS; ++s) top = __builtin_amdgcn_mfma_i32_16x16x64_i8(key[s], q[t][PARTS - 1][j % R][s], top, 0, 0, 0);
            acc += top << 7;
        }
        return acc;
    };

    // the same without b from rows that were fetched for sweep 1: registers 2 and 3 are the rows with exchanged halves
    auto tile_scores1 = [&](const v4i (&buf)[NSB][STEPS], int j, int t) -> v4i {
        v4i acc = tile_scores(buf, j, t, 0);
        if constexpr (TWIST) {
            v4i x = __builtin_amdgcn_mfma_i32_16x16x64_i8(buf[j / R][0], qx[t][0], v4i{0, 0, 0, 0}, 0, 0, 0);
            if (GROUP) x += __builtin_amdgcn_mfma_i32_16x16x64_i8(buf[j / R][0], qx[t][PARTS - 1], v4i{0, 0, 0, 0}, 0, 0, 0) << 7;
            acc[2] = x[2];
            acc[3] = x[3];
        }
        return acc;
    };

    int nv = max(0, min(L - h * Lr, Lr));                          // real keys of this lane's range
    const int nv_all = max(0, min(L - (4 * wv + 3) * Lr, Lr));     // of the wavefront's last range: the fewest

    // ---- sweep 1: bucket maxima --------------------------------------------------------------------------------------
    // A range of one group (NWM == 1) keeps every score; else tiles j and j + PAIR share a bucket, and so do all groups (of
    // the same parity, if there are 32): two scores per v_max3.
    int bm[UT][NB];
#pragma unroll
    for (int t = 0; t < UT; ++t)
#pragma unroll
        for (int b = 0; b < NB; ++b) bm[t][b] = INT32_MIN;
    auto maxima = [&](const v4i (&buf)[NSB][STEPS], int w, auto par, auto half, auto masked) {
        constexpr int PAR = decltype(par)::value, J0 = decltype(half)::value * TB;
#pragma unroll
        for (int t = 0; t < UT; ++t)
#pragma unroll
            for (int jb = 0; jb < TB; jb += 2 * PAIR)
#pragma unroll
                for (int e = 0; e < PAIR; ++e) {
                    const int j = jb + e;
                    v4i x = tile_scores1(buf, j, t), y = tile_scores1(buf, j + PAIR, t);
                    if (decltype(masked)::value) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            x[i] = mask_beyond(x[i], 32 * w + 4 * (J0 + j) + i, nv);
                            y[i] = mask_beyond(y[i], 32 * w + 4 * (J0 + j + PAIR) + i, nv);
                        }
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if (NWM == 1) {
                            bm[t][(4 * (J0 + j) + i) % NB] = x[i];
                            bm[t][(4 * (J0 + j + PAIR) + i) % NB] = y[i];
                        } else {
                            int &m = bm[t][(NB == 32 ? 16 * PAR : 0) + 4 * ((J0 + jb) / 2 + e) + i];
                            m = max(max(x[i], y[i]), m);
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
    };
    {
        auto group = [&](int w, auto par, auto masked) {
            constexpr int PAR = decltype(par)::value;
            auto batch = [&](auto half) {
                constexpr int HB = decltype(half)::value, P = BPG == 1 ? PAR : HB & 1;
                request(rows[P ^ 1], w * BPG + HB + 1, twisted);
                maxima(rows[P], w, par, half, masked);
            };
            batch(std::integral_constant<int, 0>{});
            if constexpr (BPG >= 2) batch(std::integral_constant<int, 1>{});
            if constexpr (BPG == 4) {
                batch(std::integral_constant<int, 2>{});
                batch(std::integral_constant<int, 3>{});
            }
        };
        const std::integral_constant<int, 0> even{};
        const std::integral_constant<int, 1> odd{};
        if (NWM == 1) {
            if (nv_all >= 32) group(0, even, std::false_type{});
            else group(0, even, std::true_type{});
        } else {
            // (one loop without and one with the test for real keys: with both in one body the buckets changed registers, 32 moves for
            // every 48 instructions that do something)
            int w = 0;
            for (; 32 * (w + 2) <= nv_all; w += 2) {
                group(w, even, std::false_type{});
                group(w + 1, odd, std::false_type{});
            }
            for (; w < NW; w += 2) {
                group(w, even, std::true_type{});
                if (w + 1 < NW) group(w + 1, odd, std::true_type{});
            }
        }
    }
    request(rows[0], 0, voff);   // sweep 2 starts with what is on its way during the bounds

    // ---- bounds -------------------------------------------------------------------------------------------------------
    // The histogram's bins lie in a window around the thresholds (split_window); what is above goes to the last bin, what is below it, an empty
    // bucket too, to a word of the lane before the bins (mostly: most maxima are, and would otherwise meet in one).  Bins over all
    // maxima, three times the distance from the smallest to the mean, were two to six times as wide and the band half as long again:
    // N = 16, L = 4096, k = 32, keep = 205 72 keys of a unit instead of 54, the mask 103 -> 97 us.
    // (Empty buckets without a branch each: that took the bounds of a wavefront that has some, for which the others wait, from 6 k to 12 k
    // cycles of 48 k.)
    const bool full = nv_all >= 32, none = 4 * wv * Lr >= L;
    {
        float *s_sum = reinterpret_cast<float *>(s_toth);
#pragma unroll
        for (int t = 0; t < UT; ++t) {
            int mn = INT32_MAX, all = 0;                 // 32 scores below 2^24 each
            if (NWM > 1 || full) {
                unsigned sum_of = 0;
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    mn = min(mn, bm[t][b]);
                    sum_of += (unsigned)bm[t][b];
                }
                all = (int)sum_of;
                // (a range that ends beyond the head has buckets of fewer keys or of none: their maxima are lower)
                if (NWM > 1 && nv < Lr) {
                    mn = INT32_MAX;
                    all = 0;
                }
            } else if (!none) {
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    const bool real = bm[t][b] != INT32_MIN;
                    mn = real ? min(mn, bm[t][b]) : mn;
                    all += real ? bm[t][b] : 0;
                }
            }
            float sum = (float)all;
            Halves a = row_halves(mn), b = wave_halves(min(a.lower, a.upper));
            mn = min(b.lower, b.upper);
            a = row_halves(__float_as_int(sum));
            b = wave_halves(__float_as_int(__int_as_float(a.lower) + __int_as_float(a.upper)));
            sum = __int_as_float(b.lower) + __int_as_float(b.upper);
            if (g == 0) {
                s_totl[wv * U + kTile * t + c] = mn;
                s_sum[wv * U + kTile * t + c] = sum;
            }
        }
        __syncthreads();
        // maxima that were added up: NB per full range, or every key
        const int added = NWM == 1 ? min(L, 32 * 4 * W) : NB * (L / Lr);
        SplitBins bins[UT];
        bool open[UT];                                   // thresholds to be looked for
#pragma unroll
        for (int t = 0; t < UT; ++t) {
            int mn = INT32_MAX;
            float sum = 0.f;
#pragma unroll 4
            for (int x = 0; x < W; ++x) {
                mn = min(mn, s_totl[x * U + kTile * t + c]);
                sum += s_sum[x * U + kTile * t + c];
            }
            bins[t] = window_bins(sum / (float)added, mn, a.low, a.high, !AGAIN);
            open[t] = true;
            if (wv == 0 && g == 0) s_need[kTile * t + c] = mn;
        }
        // A threshold that lies outside of the window (SplitPlan) is looked for on the other side of it, in another histogram over what is left between
        // the ends of all maxima and the threshold that was found.  That takes a workgroup 2 to 3 us; sweeps of the keys, which would find it too: keys in eight
        // clusters, N = 16, L = 8192, k = 64, keep = 82, groups of 8 156 -> 57 us, N = 4, L = 16384, keep = 164 1080 -> 376 (with bins over all maxima, which have
        // long bands there, 73 and 520), log-normal norms, N = 16, L = 4096, k = 32, keep = 410 138 -> 111 (121).
        for (int round = 1;; ++round) {
#pragma unroll
            for (int t = 0; t < UT; ++t) {
                unsigned *uh = hist + (kTile * t + c) * kBinStride + kBelow;
                if (!none && open[t]) {
#pragma unroll
                    for (int b = 0; b < NB; ++b) atomicAdd(&uh[max(split_bin(bins[t], bm[t][b]), -1 - g)], 1u);
                }
                if (wv == 0 && g == 0) {
                    s_base[kTile * t + c] = bins[t].base;
                    s_shift[kTile * t + c] = bins[t].shift;
                }
            }
            __syncthreads();
            // 16 lanes per unit, 8 bins each: th is the lowest bin edge that at most target_h maxima reach, tl the highest
            // that at least target_l reach
            for (int b4 = wv; b4 < 4 * UT; b4 += W) {
                const int u = 4 * b4 + g;
                v4i *uh = reinterpret_cast<v4i *>(hist + u * kBinStride + kBelow + 8 * c);
                const v4i x = uh[0], y = uh[1];
                const int in[8] = {x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]};
                const int beyond = row_sum_above(((in[0] + in[1]) + (in[2] + in[3])) + ((in[4] + in[5]) + (in[6] + in[7])));
                int edge_h = kBins, edge_l = -1;         // in this lane: lowest edge with suffix <= target_h, highest with >= target_l
                int suffix = beyond;
#pragma unroll
                for (int e = 7; e >= 0; --e) {
                    suffix += in[e];                      // maxima in bins >= 8 c + e
                    if (suffix <= a.target_h) edge_h = 8 * c + e;
                    if (suffix >= a.target_l && edge_l < 0) edge_l = 8 * c + e;
                }
                // how many of them reach the edges
                auto reach_low = [&] {
                    int n = INT32_MAX, s = beyond;
#pragma unroll
                    for (int e = 7; e >= 0; --e) {
                        s += in[e];
                        n = s >= a.target_l ? min(n, s) : n;
                    }
                    return -row_max(-n);
                };
                auto reach_high = [&] {
                    int n = 0, s = beyond;
#pragma unroll
                    for (int e = 7; e >= 0; --e) {
                        s += in[e];
                        n = s <= a.target_h ? s : n;
                    }
                    return row_max(n);
                };
                edge_h = -row_max(-edge_h);
                edge_l = row_max(edge_l);
                const SplitBins now = {s_base[u], s_shift[u]};
                const bool below = edge_l < 0, above = edge_h == kBins;
                int tl = now.base + (max(edge_l, 0) << now.shift), th = now.base + (edge_h << now.shift), flags = 0;
                if (round == 1) {
                    if (below) tl = s_need[u];                                                // the smallest maximum
                    if (above) th = (GROUP ? a.vec : 1) * k * 16384 + 1;                      // above every score
                    if (AGAIN && __ballot(below || above) != 0) {
                        const int low = reach_low(), between = (below ? added : low) - reach_high();
                        if (split_crowded(between, a.target_l, a.target_h)) flags = (below ? 1 : 0) | (above ? 2 : 0);
                    }
                } else {
                    // (as long as it helps: the bracket gets shorter, and has bins of more than one score)
                    const bool shorter = now.shift > 0 && th - tl <= kBins / 4 << now.shift, was = s_nb[u] != 0;
                    const int between = reach_low() - reach_high();
                    if (was && !below && round < kBinRounds && shorter && split_crowded(between, a.target_l, a.target_h)) flags = 4;
                    if (!was) { tl = s_tl[u]; th = s_th[u]; }
                }
                if (AGAIN && __ballot(flags != 0) != 0) {          // (all 16 lanes of a unit have read; the other units are not looked at again)
                    uh[0] = uh[1] = v4i{0, 0, 0, 0};
                }
                if (c == 0) {
                    s_tl[u] = tl;
                    s_th[u] = th;
                    if (AGAIN) s_nb[u] = flags;
                }
            }
            __syncthreads();
            if constexpr (!AGAIN) break;
            int flags[UT], any = 0;
#pragma unroll
            for (int t = 0; t < UT; ++t) any |= flags[t] = s_nb[kTile * t + c];
            // every wavefront sees all units: the same outcome everywhere
            if (__ballot(any != 0) == 0) break;
            if (round == 1) {
                // the ends of all maxima, those of ranges that end beyond the head too
#pragma unroll
                for (int t = 0; t < UT; ++t) {
                    int least = INT32_MAX, most = INT32_MIN;
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        asm volatile("" : "+v"(bm[t][b]));           // (not computed ahead of the loop)
                        least = min(least, bm[t][b] != INT32_MIN ? bm[t][b] : INT32_MAX);
                        most = max(most, bm[t][b]);
                    }
                    Halves x = row_halves(least), y = wave_halves(min(x.lower, x.upper));
                    least = min(y.lower, y.upper);
                    x = row_halves(most), y = wave_halves(max(x.lower, x.upper));
                    most = max(y.lower, y.upper);
                    if (g == 0) {
                        s_totl[wv * U + kTile * t + c] = least;
                        s_toth[wv * U + kTile * t + c] = most;
                    }
                }
                __syncthreads();
            }
#pragma unroll
            for (int t = 0; t < UT; ++t) {
                int lo = s_tl[kTile * t + c], hi = s_th[kTile * t + c];
                open[t] = flags[t] != 0;
                if (flags[t] & 1) {
                    lo = INT32_MAX;
                    for (int x = 0; x < W; ++x) lo = min(lo, s_totl[x * U + kTile * t + c]);
                }
                if (flags[t] & 2) {
                    hi = INT32_MIN;
                    for (int x = 0; x < W; ++x) hi = max(hi, s_toth[x * U + kTile * t + c] + 1);
                }
                bins[t] = bracket_bins(lo, hi);
            }
        }
    }

    // ---- sweep 2: bitmaps of score >= tl and score >= th, until every unit's bracket is good ---------------------------
    // (the largest product of two codes is -128 * -128, the smallest -128 * 127: with thresholds between these ends no difference reaches 2^24)
    const int smax = (GROUP ? a.vec : 1) * k * 16384, smin = -(GROUP ? a.vec : 1) * k * 16256;
    SplitBracket br[UT];
#pragma unroll
    for (int t = 0; t < UT; ++t) {
        const int tl = s_tl[kTile * t + c];
        br[t] = {tl, min(max(s_th[kTile * t + c], tl + 1), smax + 1), smin, smax + 1, L, 0};
    }
    // The keys at or above th go to LDS, where the histogram was, and those that are kept of the band, which the registers have, join them there:
    // half the registers of two bitmaps, and nothing to clear or to merge.
    unsigned *sel = hist;                          // [U][at.sel]
    unsigned *mine_at[UT];
#pragma unroll
    for (int t = 0; t < UT; ++t) mine_at[t] = sel + (kTile * t + c) * at.sel + h * NW;
    unsigned band[UT][NWM];
    int nl[UT], nh[UT], band0[UT];                 // counts of the unit; band keys in the ranges before this lane's
    const SignMasks signs;
    for (int tries = 0;; ++tries) {
        int cl[UT], ch[UT];
#pragma unroll
        for (int t = 0; t < UT; ++t) cl[t] = ch[t] = 0;
        // the sweep's masks and addresses are the same in every round: computed ahead for all words they would fill the registers, so the
        // compiler is kept from seeing it
        asm volatile("" : "+v"(nv), "+s"(batches));
#pragma unroll
        for (int w = 0; w < NWM; ++w) {
#pragma unroll
            for (int t = 0; t < UT; ++t) band[t][w] = 0u;
            if (w < NW) {
                unsigned wl[UT], wh[UT], sl[UT][4], sh[UT][4];
#pragma unroll
                for (int t = 0; t < UT; ++t) wl[t] = wh[t] = 0u;
#pragma unroll
                for (int hb = 0; hb < BPG; ++hb) {
                    const int P = BPG == 1 ? w & 1 : hb & 1;
                    request(rows[P ^ 1], w * BPG + hb + 1, voff);
#pragma unroll
                    for (int j = 0; j < TB; ++j)
#pragma unroll
                        for (int t = 0; t < UT; ++t) {
                            const v4i x = tile_scores(rows[P], j, t, -br[t].tl);
                            v4i y;
#pragma unroll
                            for (int i = 0; i < 4; ++i) y[i] = x[i] - (br[t].th - br[t].tl);
                            if constexpr (COPIES) {
                                signs.tile(sl[t], 4 * (hb * TB + j), x);
                                signs.tile(sh[t], 4 * (hb * TB + j), y);
                            } else {
                                shift_in_signs(wl[t], x);
                                shift_in_signs(wh[t], y);
                            }
                            if (j % 2 == 1) __builtin_amdgcn_sched_barrier(0);      // else every tile's scores live at once
                        }
                }
#pragma unroll
                for (int t = 0; t < UT; ++t) {
                    wl[t] = ~(COPIES ? SignMasks::word(sl[t]) : __brev(wl[t]));             // (shifted in: the first key of the word first)
                    wh[t] = ~(COPIES ? SignMasks::word(sh[t]) : __brev(wh[t]));
                }
                if (32 * (w + 1) > nv_all) {
                    const int left = nv - 32 * w;                        // real keys of this word
                    const unsigned real = left >= 32 ? ~0u : left <= 0 ? 0u : (1u << left) - 1u;
#pragma unroll
                    for (int t = 0; t < UT; ++t) {
                        wl[t] &= real;
                        wh[t] &= real;
                    }
                }
#pragma unroll
                for (int t = 0; t < UT; ++t) {
                    cl[t] += __popc(wl[t]);
                    ch[t] += __popc(wh[t]);
                    band[t][w] = wl[t] & ~wh[t];
                    mine_at[t][w] = wh[t];
                }
            }
        }
        request(rows[0], 0, voff);
#pragma unroll
        for (int t = 0; t < UT; ++t) {
            // (count(>= tl) << 16 | count(>= th)) of the unit's ranges in this wavefront: at most 8192 each
            const int mine = cl[t] << 16 | ch[t];
            int all;
            const int before = unit_excl_scan(mine, g, &all);
            band0[t] = (before >> 16) - (before & 0xffff);
            if (g == 0) s_totl[wv * U + kTile * t + c] = all;
        }
        __syncthreads();
        bool again = false;
#pragma unroll
        for (int t = 0; t < UT; ++t) {
            nl[t] = nh[t] = 0;
#pragma unroll 4
            for (int x = 0; x < W; ++x) {
                const int v = s_totl[x * U + kTile * t + c];
                const int vl = v >> 16, vh = v & 0xffff;
                nl[t] += vl;
                nh[t] += vh;
                band0[t] += x < wv ? vl - vh : 0;
            }
            if (!br[t].good(nl[t], nh[t], keep, kBandCap)) {
                again = true;
                br[t].move(nl[t], nh[t], keep, kBandCap, tries);
            }
        }
        // every wavefront sees all units: the same outcome everywhere
        if (__ballot(again) == 0) break;
        __syncthreads();
    }

    // ---- band list: keys between the thresholds, in key order -----------------------------------------------------------
    // A unit whose bracket is one score value wide takes its first keys of that value and needs no scores.
    bool scored[UT];
#pragma unroll
    for (int t = 0; t < UT; ++t) {
        scored[t] = nh[t] < keep && br[t].th - br[t].tl != 1;
        uint16_t *ul = list + (kTile * t + c) * kBandCap;
        int pos = band0[t];
#pragma unroll
        for (int w = 0; w < NWM; ++w) {
            if (w < NW) {
                unsigned m = scored[t] ? band[t][w] : 0u;
                const int key1 = h * Lr + 32 * w - 1;
                while (m) {
                    ul[pos++] = (uint16_t)(key1 + __ffs(m));             // pos < nl - nh <= kBandCap
                    m &= m - 1u;
                }
            }
        }
        if (wv == 0 && g == 0) {
            s_tl[kTile * t + c] = br[t].tl;
            s_th[kTile * t + c] = br[t].th;
            s_need[kTile * t + c] = keep - nh[t];
            s_nb[kTile * t + c] = scored[t] ? nl[t] - nh[t] : 0;
        }
    }
    __syncthreads();

    // ---- band scores and exact threshold: 16 lanes per unit, four units at a time per wavefront -------------------------
    for (int b4 = wv; b4 < 4 * UT; b4 += W) {
        const int u = 4 * b4 + g;                 // this lane's unit here
        const int nb = s_nb[u], need = s_need[u], ulo = s_tl[u];
        const int most = max(max(__builtin_amdgcn_readlane(nb, 0), __builtin_amdgcn_readlane(nb, 16)),
                             max(__builtin_amdgcn_readlane(nb, 32), __builtin_amdgcn_readlane(nb, 48)));
        if (most == 0) continue;
        const uint16_t *ul = list + u * kBandCap;
        const unsigned char *uq = s_q + u * qstride;
        // (the loops over slots leave where the band ends: one taken branch, not one per slot that is skipped)
        int sc[kBandSlots];                        // (those behind the last slots that the band reaches are not looked at)
        // (Ranges of more than eight groups: with long lists up to 5 % faster if they are written all the same, N = 1, L = 8200, keep = 1640 94.3 and
        // 89.4 us, in one launch with the attention always, N = 16, L = 5000, keep = 250 289 and 284; by themselves with short lists 154 and 156.
        // The others are 1 to 3 % slower: N = 16, L = 4096, keep = 205 98.8 and 101.)
        if (NWM == 16) {
#pragma unroll
            for (int i = 0; i < kBandSlots; ++i) sc[i] = INT32_MIN;
        }
        int peak = INT32_MIN;
        const bool two = NWM == 1 && most <= 32;   // of the first slots: where every key is its own bucket a band is one bin of the histogram
#pragma unroll
        for (int i0 = 0; i0 < kBandSlots; i0 += SG) {
            if (16 * i0 >= most) break;
            int s[SG], sh[SG];
            if constexpr (LPK > 1) {
                // a row's pieces by neighbouring lanes, whose sums for the LPK entries of their group change places in the end
                const int8_t *kr[SG][LPK];
                const int p = 16 * (c & (LPK - 1));
#pragma unroll
                for (int i = 0; i < SG; ++i) {
                    const uint16_t *entries = ul + (c & ~(LPK - 1)) + 16 * (i0 + i);      // (behind the band: some key, whose score is not used)
#pragma unroll
                    for (int j = 0; j < LPK; ++j) kr[i][j] = Kh + min((unsigned)entries[j], (unsigned)(L - 1)) * (unsigned)k + p;
                }
                const v4i ql = *reinterpret_cast<const v4i *>(uq + p), qh = *reinterpret_cast<const v4i *>(uq + (GROUP ? k + 16 : 0) + p);
                constexpr int AT = LPK == 2 ? SG : 2;            // slots whose rows are requested together: 32 registers
#pragma unroll
                for (int i1 = 0; i1 < SG; i1 += AT) {
                    v4i kk[AT][LPK];
#pragma unroll
                    for (int i = 0; i < AT; ++i)
#pragma unroll
                        for (int j = 0; j < LPK; ++j) kk[i][j] = *reinterpret_cast<const v4i *>(kr[i1 + i][j]);
#pragma unroll
                    for (int i = 0; i < AT; ++i) {
                        int part[LPK];
#pragma unroll
                        for (int j = 0; j < LPK; ++j) {
                            int top = 0;
                            part[j] = 0;
#pragma unroll
                            for (int x = 0; x < 4; ++x) {
                                part[j] = __builtin_amdgcn_sdot4(ql[x], kk[i][j][x], part[j], false);
                                if (GROUP) top = __builtin_amdgcn_sdot4(qh[x], kk[i][j][x], top, false);
                            }
                            if (GROUP) part[j] += 128 * top;
                        }
                        s[i1 + i] = key_sums<LPK>(part, lane);
                        sh[i1 + i] = 0;
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {
                const int8_t *kr[SG];
#pragma unroll
                for (int i = 0; i < SG; ++i) {
                    if (i >= 2 && two) continue;
                    kr[i] = Kh + min((unsigned)ul[c + 16 * (i0 + i)], (unsigned)(L - 1)) * (unsigned)k;      // (behind the band: some key, whose score is not used)
                    s[i] = sh[i] = 0;
                }
                auto piece = [&](int p) {
                    v4i kk[SG];
#pragma unroll
                    for (int i = 0; i < SG; ++i) if (i < 2 || !two) kk[i] = *reinterpret_cast<const v4i *>(kr[i] + 16 * p);
                    const v4i ql = *reinterpret_cast<const v4i *>(uq + 16 * p);
                    const v4i qh = *reinterpret_cast<const v4i *>(uq + (GROUP ? k + 16 : 0) + 16 * p);
#pragma unroll
                    for (int i = 0; i < SG; ++i)
#pragma unroll
                        for (int x = 0; x < 4; ++x) {
                            if (i >= 2 && two) continue;
                            s[i] = __builtin_amdgcn_sdot4(ql[x], kk[i][x], s[i], false);
                            if (GROUP) sh[i] = __builtin_amdgcn_sdot4(qh[x], kk[i][x], sh[i], false);
                        }
                    if (NWM == 1 || K == 0 || K > 32) __builtin_amdgcn_sched_barrier(0);       // the rows of four keys do not fit the registers
                };
                if constexpr (K != 0 && (NWM > 1 || K <= 64)) {        // (128 in a row: 80 to 504 registers through scratch)
#pragma unroll
                    for (int p = 0; p < K / 16; ++p) piece(p);
                } else {
#pragma unroll 1
                    for (int p = 0; p < k / 16; ++p) piece(p);
                }
            }
#pragma unroll
            for (int i = 0; i < SG; ++i) {
                if (i >= 2 && two) {
                    sc[i0 + i] = INT32_MIN;
                    continue;
                }
                const int v = s[i] + 128 * sh[i];
                sc[i0 + i] = c + 16 * (i0 + i) < nb ? v : INT32_MIN;
                peak = max(peak, sc[i0 + i]);
            }
        }
        auto keep_key = [&](unsigned key) { atomicOr(&sel[u * at.sel + (key >> 5)], 1u << (key & 31)); };
        if constexpr (NWM == 1) {                  // (bands of single keys: a few of them, mostly)
            if (most <= 16) {
                // One key to a lane: kept if fewer than `need` others come before it (|scores| < 2^25; the lower key first among equals).
                // No search, whose cuts wait for each other: N = 2, L = 256, k = 16, keep = 26, both launches 11.1 -> 9.4 us in a graph, N = 192,
                // L = 256, keep = 20 41.9 -> 38.1.
                const int mine = c < nb ? 16 * sc[0] + 15 - c : INT32_MIN;
                int before = 0;
                auto against = [&](auto r) { before += __builtin_amdgcn_update_dpp(0, mine, 0x120 + decltype(r)::value /* row_ror */, 0xF, 0xF, true) > mine; };
                against(std::integral_constant<int, 1>{}); against(std::integral_constant<int, 2>{}); against(std::integral_constant<int, 3>{});
                against(std::integral_constant<int, 4>{}); against(std::integral_constant<int, 5>{}); against(std::integral_constant<int, 6>{});
                against(std::integral_constant<int, 7>{}); against(std::integral_constant<int, 8>{}); against(std::integral_constant<int, 9>{});
                against(std::integral_constant<int, 10>{}); against(std::integral_constant<int, 11>{}); against(std::integral_constant<int, 12>{});
                against(std::integral_constant<int, 13>{}); against(std::integral_constant<int, 14>{}); against(std::integral_constant<int, 15>{});
                if (c < nb && before < need) keep_key(ul[c]);
                continue;
            }
        }
        // The need-th largest of the band: all its scores are >= tl and at least need of them exist.  The interval is cut
        // where it would be cut for evenly spread scores, every third time in the middle, until a cut leaves exactly need.
        int lo_ = ulo, hi_ = nb ? max(row_max(peak), ulo) : ulo, cnt_lo = nb, cnt_hi = 0;   // counts >= lo_ and > hi_
        for (int cut = 0; __ballot(lo_ < hi_) != 0; cut = cut == 2 ? 0 : cut + 1) {
            const int width = hi_ - lo_;                  // |scores| < 2^27
            int step = (width + 1) >> 1;
            if (cut < 2)
                step = min(max((int)((float)width * (float)(cnt_lo - need) * __builtin_amdgcn_rcpf((float)(cnt_lo - cnt_hi))), 1), width);
            const int mid = lo_ + step;
            int cnt = 0;
#pragma unroll
            for (int i0 = 0; i0 < kBandSlots; i0 += SG) {
                if (16 * i0 >= most) break;
#pragma unroll
                for (int i = 0; i < SG; ++i) cnt += sc[i0 + i] >= mid;
            }
            cnt = row_sum(cnt);
            if (lo_ < hi_) {
                const bool ge = cnt >= need;
                lo_ = ge ? mid : lo_;
                cnt_lo = ge ? cnt : cnt_lo;
                hi_ = !ge ? mid - 1 : cnt == need ? mid : hi_;
                cnt_hi = ge ? cnt_hi : cnt;
            }
        }
        const int Tx = lo_;
        if (__ballot(nb && cnt_lo != need) == 0) {        // no tie at the threshold is left out: no order among them
#pragma unroll
            for (int i0 = 0; i0 < kBandSlots; i0 += SG) {
                if (16 * i0 >= most) break;
                unsigned key[SG];
#pragma unroll
                for (int i = 0; i < SG; ++i) key[i] = ul[c + 16 * (i0 + i)];
#pragma unroll
                for (int i = 0; i < SG; ++i)
                    if (sc[i0 + i] >= Tx) keep_key(key[i]);
            }
            continue;
        }
        int gt = 0;
#pragma unroll
        for (int i0 = 0; i0 < kBandSlots; i0 += SG) {
            if (16 * i0 >= most) break;
#pragma unroll
            for (int i = 0; i < SG; ++i) gt += sc[i0 + i] > Tx;
        }
        const int need_eq = need - row_sum(gt);
        int eq_before = 0;
        const unsigned below = (1u << c) - 1u;
#pragma unroll
        for (int i = 0; i < kBandSlots; ++i) {
            if (16 * i >= most) break;
            const bool eq = sc[i] == Tx && c + 16 * i < nb;
            const unsigned meq = (unsigned)(__ballot(eq) >> (16 * g)) & 0xffffu;
            const bool take = c + 16 * i < nb && (sc[i] > Tx || (eq && eq_before + __popc(meq & below) < need_eq));
            eq_before += __popc(meq);
            if (take) keep_key(ul[c + 16 * i]);
        }
    }
    __syncthreads();

    // ---- emission -----------------------------------------------------------------------------------------------------
    unsigned words[UT][NWM];                       // the lists as bitmaps
    int out0[UT];
#pragma unroll
    for (int t = 0; t < UT; ++t) {
        const bool tie = nh[t] < keep && !scored[t];
        int quota = max(0, keep - nh[t] - band0[t]);                 // ties this lane may still keep
        int mine = 0;
#pragma unroll
        for (int w = 0; w < NWM; ++w) {
            words[t][w] = 0u;
            if (w < NW) {
                words[t][w] = mine_at[t][w];
                if (tie) {
                    const unsigned more = lowest_set_bits(band[t][w], quota);
                    quota -= __popc(more);
                    words[t][w] |= more;
                }
                mine += __popc(words[t][w]);
            }
        }
        int all;
        out0[t] = unit_excl_scan(mine, g, &all);
        if (g == 0) s_totl[wv * U + kTile * t + c] = all;
    }
    __syncthreads();
    uint16_t *image = reinterpret_cast<uint16_t *>(lds + at.hist);      // [U * keep]; everything there is dead
    int32_t *out = a.idx + ((size_t)n * G + u0) * keep;
#pragma unroll
    for (int t = 0; t < UT; ++t) {
#pragma unroll 4
        for (int x = 0; x < wv; ++x) out0[t] += s_totl[x * U + kTile * t + c];
        const bool live = kTile * t + c < nu;
        int pos = (kTile * t + c) * keep + out0[t];
#pragma unroll
        for (int w = 0; w < NWM; ++w) {
            if (w < NW) {
                unsigned m = live ? words[t][w] : 0u;
                const int key1 = h * Lr + 32 * w - 1;
                if (!a.direct) {
                    while (m) {
                        image[pos++] = (uint16_t)(key1 + __ffs(m));
                        m &= m - 1u;
                    }
                } else {
                    while (m) {
                        out[pos++] = key1 + __ffs(m);
                        m &= m - 1u;
                    }
                }
            }
        }
    }
    if (a.direct) return;
    __syncthreads();
    const int total = nu * keep;
    for (int e = 4 * tid; e < total; e += 4 * T) {
        const uint2 four = *reinterpret_cast<const uint2 *>(image + e);
        const int v[4] = {(int)(four.x & 0xffffu), (int)(four.x >> 16), (int)(four.y & 0xffffu), (int)(four.y >> 16)};
        if (e + 4 <= total) {
            *reinterpret_cast<int4 *>(out + e) = make_int4(v[0], v[1], v[2], v[3]);
        } else {
            for (int i = 0; e + i < total; ++i) out[e + i] = v[i];
        }
    }

    // ---- attention over the lists -------------------------------------------------------------------------------------
    if constexpr (ATTEND != kNoAttend) {
        unsigned *room = reinterpret_cast<unsigned *>(lds + at.attend);     // behind the image: nobody else reads or writes there any more
        const int vec = GROUP ? a.vec : 1;
        if constexpr (ATTEND == kAttendTile) {
            static_assert(UT == 1, "one tile of units");
            const size_t head = (size_t)n * L * 64;
            const uint16_t *Q = static_cast<const uint16_t *>(a.attend.Q) + head, *Kx = static_cast<const uint16_t *>(a.attend.K) + head,
                           *V = static_cast<const uint16_t *>(a.attend.V) + head;
            // (from where the image was: the lists are in memory, and the bitmaps still in the registers)
            char *tile = reinterpret_cast<char *>(image);
            const int total = union_entries<NWM>(words[0], NW, h * Lr, c < nu, reinterpret_cast<unsigned *>(tile + TileLds(W, a.attend.most).list), s_totl);
            if (!attend_tile(Q + (size_t)u0 * 64, Kx, V, a.attend.O + head + (size_t)u0 * 64, nu, total, a.attend.scale, a.attend.most, tile))
                attend_listed(a.attend, out, tile, L, keep, n, u0, nu);
        } else if constexpr (GROUP && ATTEND == kAttendBf16) {
            attend_block_units<64>(a.attend, image, reinterpret_cast<char *>(room), L, keep, vec, n, u0, nu);
        } else {
            typedef std::conditional_t<ATTEND == kAttendF32, float, uint16_t> T;
            if (a.attend.d == 64) attend_block<T, 64>(a.attend, image, room, L, keep, vec, n, u0, nu, W);
            else attend_block<T, 128>(a.attend, image, room, L, keep, vec, n, u0, nu, W);
        }
    }
}

// ---- host side -----------------------------------------------------------------------------------------------------------

inline size_t attend_lds_bytes(const dsa_shape &sh, int W, int pad)
{
    if (sh.vec > 1 && sh.dtype == DSA_BF16) return (size_t)W * (unit_tile_bytes<64>() + pad * sizeof(unsigned));
    return (size_t)W * (sh.dtype == DSA_F32 ? attend_rows_at_once<float>() : attend_rows_at_once<uint16_t>()) * pad * sizeof(unsigned);
}

// Whether the workgroups that make the lists attend over them too.  One launch less, lists that need not come back from memory,
// and while some workgroups select (vector issue) others gather (L2): N = 16, L = 4096, keep = 205, bf16, k = 32 232 -> 195 us.
// Both launches are better (times of two launches and of one):
//   - if few workgroups have many bytes to gather, where the rows by themselves spread over more CUs.  Single rows: up to 16 KB per
//     wavefront N = 2, L = 128, keep = 13 11.8 and 11.3; 26 KB, N = 1, L = 512, keep = 51 9.0 and 10.4, fp32, N = 2, L = 256, keep = 26, 9.2 and 9.5, N = 4, L = 256 9.2 and
//     9.6 (in a graph; N = 3, L = 200, keep = 20 10.0 and 9.8, N = 12, L = 128, keep = 13 8.9 and 8.7); 53 KB, fp32, d = 128, N = 4, L = 512, keep = 26, 12.6 and 14.1.  From 2048 wavefronts on: N = 16, L = 512, keep = 51
//     16.6 and 15.3.
//   - fp32 rows of groups, 16 or 32 to a wavefront, if the last round of workgroups leaves places of the chip idle for long: if the
//     share of the idle places, times the bytes of a wavefront, is above 20 KB per round.  Groups of 8, k = 32: N = 60, L = 552, d = 128,
//     keep = 39 (2400 wavefronts) 58.4 and 91.9, N = 8, L = 4448, keep = 94 (2240) 82.0 and 114, N = 191, L = 416, keep = 30 (3056) 59.2
//     and 66.9, k = 16, N = 113, L = 1216, keep = 17 (4520) 90.5 and 97.8; within it groups of 4, N = 65, L = 692, keep = 7 (2860) 33.2 and
//     28.8, groups of 8, k = 64, N = 127, L = 952, keep = 17 (4064) 79.3 and 73.4, k = 32, N = 32, L = 8192, keep = 82 (8192) 474 and 410.
//     (300 shapes from 1024 wavefronts on: 0.8 % behind the better of the two on average; the worst, N = 232, L = 392, keep = 19, 57.7 and 65.8.)
//   - units of several rows in bf16, if there are fewer than 2048 wavefronts or three tenths of the places are idle: groups of 4, k = 16,
//     N = 108, L = 264, keep = 14 (2160) 20.1 and 22.1, k = 48, N = 103, L = 664, keep = 40 (4532) 48.6 and 53.7; within it k = 32, N = 128,
//     L = 512, keep = 51 36.1 and 32.4, k = 64, N = 29, L = 2128, keep = 62 (3944) 58.0 and 53.3; groups of 8, k = 32: N = 32, L = 8192,
//     keep = 82 159.7 and 149.0, N = 8, L = 16384, keep = 164 147.8 and 145.1, N = 4, L = 4096, keep = 82 (1024) 23.2 and 24.4.  (200 shapes:
//     0.6 % behind the better of the two on average; lost are a few like N = 32, L = 5120, keep = 256 (5120), 134.0 and 128.1.)  These are of an attention kernel whose
//     rows went through registers; it takes 5 to 20 % less by itself now, and long lists, of groups of 4 above all, have come to be better in two launches: N = 64, L = 2000, k = 16,
//     keep = 200, groups of 4 129 and 136, N = 96, L = 1024, keep = 102, groups of 4 67.9 and 69.5, groups of 8, N = 64, L = 4096, keep = 205 165 and 167; the others still in one: N = 64,
//     L = 2048, keep = 102 59.8 and 58.1, N = 16, L = 4096, keep = 205 51.7 and 49.2, N = 32, L = 8192 154 and 152, groups of 4, N = 128, L = 512 31.9 and 31.1.  Above four
//     units to a wavefront (N = 512, L = 256, keep = 26, groups of 4, 54.7 and 60.7) and at d = 128, whose registers do not fit, never;
//   - if a CU does not hold two workgroups: 16 wavefronts, N = 8, L = 16384, keep = 164 1063 and 1106, long lists, bf16, d = 128, N = 2,
//     L = 8192, keep = 1229 420 and 424, or unions of long lists, d = 64, N = 2, L = 11600, keep = 1200 373 and 469 (but N = 2, L = 16384,
//     keep = 2048 878 and 806).
// Rows over their union (tile_most) are 2048 wavefronts and more, where a wavefront's bytes do not matter.
inline bool attend_here(const dsa_shape &sh, int W, int units, long long wgs, size_t lds)
{
    if (W > 8 || lds > 80 * 1024) return false;
    const long long waves = wgs * W;
    const long long work = ((long long)sh.keep * sh.d * (sh.dtype == DSA_F32 ? 4 : 2) + 1536) * ((units * sh.vec + W - 1) / W);
    if (sh.vec == 1) return waves >= 2048 || work <= 16 * 1024;
    // wavefronts that 256 CUs hold at a time (four to a SIMD by the registers), and places that the last round leaves idle
    const long long slots = 256LL * W * std::min(16 / W, (int)(160 * 1024 / lds)), rounds = (waves + slots - 1) / slots, idle = rounds * slots - waves;
    if (sh.dtype == DSA_F32) return idle * work <= 20 * 1024 * rounds * rounds * slots;
    return sh.d == 64 && units <= 4 * W && waves >= 2048 && 10 * idle <= 3 * rounds * slots;
}

template <int K, bool GROUP, int UT, int NB, int NWM>
hipError_t launch_split_t(const dsa_shape &sh, const SplitPlan &p, const int8_t *Qt, const int8_t *Kt, int32_t *idx,
                          const AttendPtrs *attend, bool *attended, hipStream_t st)
{
    SplitAttendArgs a{};
    a.Qt = Qt; a.Kt = Kt; a.idx = idx;
    a.L = sh.L; a.k = sh.k; a.keep = sh.keep; a.vec = sh.vec;
    a.NW = p.NW;
    a.wgs_per_head = (sh.L / sh.vec + kTile * UT - 1) / (kTile * UT);
    a.target_l = p.target_l;
    a.target_h = p.target_h;
    a.low = p.low;
    a.high = p.high;
    a.direct = (size_t)kTile * UT * sh.keep * 2 > 128 * 1024;
    const SplitLds at(p.W, UT, p.NW, sh.k, GROUP, sh.keep, a.direct != 0, band_slots<GROUP, UT, NWM>());
    size_t lds = at.bytes;
    bool attends = false;
    if (attend && !a.direct) {
        const int pad = (sh.keep + kRowPad - 1) / kRowPad * kRowPad;
        const int most = !GROUP && UT == 1 ? tile_most(sh, p.W) : 0;
        const size_t all = most ? at.hist + tile_lds_bytes(sh, p.W, most) : at.attend + attend_lds_bytes(sh, p.W, pad);
        if (attend_here(sh, p.W, kTile * UT, (long long)sh.B * sh.H * a.wgs_per_head, std::max(lds, all))) {
            lds = std::max(lds, all);
            a.attend = AttendArgs{attend->Q, attend->K, attend->V, attend->O, sh.scale, sh.d, pad, most, (unsigned)(lds - at.hist)};
            attends = *attended = true;
        }
    }
    auto go = [&](auto kern, const auto &args) -> hipError_t {
        if (hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kern), lds)) return e;
        hipLaunchKernelGGL(kern, dim3((unsigned)sh.B * sh.H * a.wgs_per_head), dim3(p.W * kWave), lds, st, args);
        return hipGetLastError();
    };
    if (!attends) return go(predict_split<K, GROUP, UT, NB, NWM, kNoAttend>, static_cast<const SplitArgs &>(a));
    if (sh.dtype == DSA_F32) return go(predict_split<K, GROUP, UT, NB, NWM, kAttendF32>, a);
    if constexpr (!GROUP && UT == 1)
        if (a.attend.most) return go(predict_split<K, GROUP, UT, NB, NWM, kAttendTile>, a);
    return go(predict_split<K, GROUP, UT, NB, NWM, kAttendBf16>, a);
}

template <int K, bool GROUP>
hipError_t launch_split_g(const dsa_shape &sh, const int8_t *Qt, const int8_t *Kt, int32_t *idx, const AttendPtrs *attend,
                          bool *attended, hipStream_t st)
{
    constexpr bool pairs = split_pairs_exist(K, GROUP);
    const SplitPlan p = split_plan(sh, pairs);
    if constexpr (pairs) {
        if constexpr (K == 64 && !GROUP)     // (the others take two tiles from five words on)
            if (p.UT == 2 && p.NW <= 4) return launch_split_t<K, GROUP, 2, 16, 4>(sh, p, Qt, Kt, idx, attend, attended, st);
        if (p.UT == 2) return launch_split_t<K, GROUP, 2, 16, 8>(sh, p, Qt, Kt, idx, attend, attended, st);
    }
    if (p.NW == 1) return launch_split_t<K, GROUP, 1, 32, 1>(sh, p, Qt, Kt, idx, attend, attended, st);
    if (p.NW <= 4) return launch_split_t<K, GROUP, 1, 32, 4>(sh, p, Qt, Kt, idx, attend, attended, st);
    if (p.NW <= 8) return launch_split_t<K, GROUP, 1, 32, 8>(sh, p, Qt, Kt, idx, attend, attended, st);
    return launch_split_t<K, GROUP, 1, 32, 16>(sh, p, Qt, Kt, idx, attend, attended, st);
}

template <int K>
hipError_t launch_split_k(const dsa_shape &sh, const int8_t *Qt, const int8_t *Kt, int32_t *idx, const AttendPtrs *attend,
                          bool *attended, hipStream_t st)
{
    if (sh.vec == 1) return launch_split_g<K, false>(sh, Qt, Kt, idx, attend, attended, st);
    return launch_split_g<K, true>(sh, Qt, Kt, idx, attend, attended, st);
}

}  // namespace
}  // namespace dsa
