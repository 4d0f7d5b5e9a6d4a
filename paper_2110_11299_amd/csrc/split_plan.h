// How predict_split cuts a shape: wavefronts per workgroup, tiles of units per workgroup, bitmap words per lane.  Host code.
#pragma once

#include "dsa_internal.h"

#include <math.h>

namespace dsa {
namespace {

constexpr int kTile = 16;               // units of one matrix instruction

// Projection dimensions that have a kernel for two tiles.
constexpr bool split_pairs_exist(int k, bool group) { return k == 64 || (k == 48 && !group); }

// Whether a threshold that the first histogram does not have is looked for in a second one.  The maxima stay in registers for it, which ranges of
// one word, five wavefronts per SIMD, do not have (L = 512, k = 32, 15 more through scratch, mask 21.9 -> 27.0 us), nor groups at k = 16, with four copies of the
// unit operands (4 more, N = 64, L = 2000, groups of 4 125.3 -> 128.8 in all).
constexpr bool split_bins_again(int k, bool group, int words) { return words > 1 && !(k == 16 && group); }

struct SplitPlan { int W, NW, UT, NB, target_l, target_h; float low, high; };

// Targets.  If a share p of a unit's keys lies above a threshold, a bucket of s keys reaches it with probability
// 1 - (1 - p)^s; the number of buckets that reach it, given the number x of keys that do, has the mean D(x) below and a
// variance that is the binomial one less what x explains.  tl is put where keep + z sigma keys are expected above it,
// th where keep - z sigma are.  A unit that misses is swept again, with its workgroup.  With z = 3.5 from 8193 wavefronts on, that was one of 4000 workgroups of 16
// units, replayed on the CPU (L = 2048 to 16384, 1 to 10 %, low-rank codes, with high-norm keys, in clusters).  In up to two rounds of workgroups nothing makes up for
// one that takes longer, and z is 4.2.  Mask, 3.5 and 4.2: N = 1, L = 16384, k = 64, keep = 164 112 and 95.6 us, N = 2, L = 8192, keep = 410 57.4 and 52.2, N = 4, L = 4096, keep = 41
// 27.0 and 24.6, N = 64, L = 2048, keep = 102, groups of 8 24.2 and 23.6; 24 others are up to 2 % slower for the longer bands (N = 64, L = 2000, k = 16, groups of 4 46.0 and 46.9).
inline void split_targets(int L, int keep, int NW, int NB, double z, int *target_l, int *target_h)
{
    if (NW == 1) {                       // every key is its own bucket
        *target_l = keep;
        *target_h = keep - 1;
        return;
    }
    const int Lr = 32 * NW;
    const double p = (double)keep / L, vx = L * p * (1.0 - p);
    // one bucket size, or two (group parity), 16 of each in `ranges` full lane ranges
    const double ranges = (double)L / Lr;
    const double size[2] = {NB == 32 ? 2.0 * ((NW + 1) / 2) : 2.0 * NW, NB == 32 ? 2.0 * (NW / 2) : 0.0}, count = 16.0 * ranges;
    double binomial = 0, cov = 0;
    for (double s : size) {
        const double miss = pow(1.0 - p, s);
        binomial += count * miss * (1.0 - miss);
        cov += count * s * p * miss;
    }
    auto buckets = [&](double x) {
        const double share = fmin(fmax(x / L, 0.0), 1.0);
        double d = 0;
        for (double s : size) d += count * (1.0 - pow(1.0 - share, s));
        return d;
    };
    const double slope = vx > 0 ? fmax(cov / vx, 1e-6) : 1.0;
    const double sigma = sqrt(fmax(binomial - (vx > 0 ? cov * cov / vx : 0.0), 0.0)) / slope;
    const double reach = z * sigma + 1.0;
    int l = (int)ceil(buckets(keep + reach)), h = (int)floor(buckets(keep - reach));
    if (keep - reach < 1.0) h = 0;
    const int most = (int)(count * NB / 16);
    l = l > most ? most : l < 1 ? 1 : l;
    h = h > l - 1 ? l - 1 : h;
    *target_l = l;
    *target_h = h;
}

// Where the histogram of a unit's bucket maxima has its bins: from mean + low * reach to mean + high * reach, reach being the distance from the
// smallest maximum to the mean.  The place of the maximum that a given share of them reaches lies within the tables, if the codes are of low
// rank: they are its 0.2 and 99.8 % quantiles over units, the lowest and highest of them over heads (rank 8 to 64, k = 16 to 64, L = 256 to 16384,
// single rows and groups of 8, high-norm keys from L = 1024 on), and a little beyond.  Keys whose norms vary more, or that lie in clusters, put it
// elsewhere: a few of them move the smallest maximum or the mean.
//   Otherwise the window is three quarters of the reach wide at least, and where a threshold lies outside of it, a second histogram
//   has it (predict_split).  Keys of a band, by the tables alone, so, and with bins over all maxima: L = 4096, keep = 205 52, 54 and 71.
//   No second histogram (once): the window is 1.75 times the reach wide, where 3 cover nearly all maxima, and starts a third of it below the tables.  The longest band of four
//   units at L = 512, keep = 51, by the tables alone, so, and over all maxima: 4.7, 9.3 and 14.4 keys (up to 16 are put in order without a search), 5 % of keys with four times
//   the norm 169, 19 and 32, log-normal norms 254, 15 and 28, keys in eight clusters 35, 13 and 21.
inline void split_window(int buckets, bool once, int target_l, int target_h, float *low, float *high)
{
    constexpr int N = 17;
    constexpr double share[N] = {0.0, 0.005, 0.015, 0.03, 0.05, 0.08, 0.125, 0.175, 0.25, 0.35, 0.45, 0.55, 0.65, 0.75, 0.85, 0.93, 1.0};
    constexpr double lowest[N] = {0.40, 0.40, 0.40, 0.36, 0.30, 0.24, 0.20, 0.14, 0.06, -0.07, -0.13, -0.30, -0.46, -0.55, -0.75, -1.0, -1.0};
    constexpr double highest[N] = {1.9, 1.6, 1.5, 1.5, 1.15, 0.95, 0.82, 0.62, 0.50, 0.30, 0.20, 0.06, -0.03, -0.10, -0.15, -0.25, -0.35};
    auto at = [&](const double (&y)[N], double x) {
        int i = 1;
        while (i < N - 1 && share[i] < x) ++i;
        return y[i - 1] + (y[i] - y[i - 1]) * fmin((x - share[i - 1]) / (share[i] - share[i - 1]), 1.0);
    };
    double lo = at(lowest, (double)target_l / buckets), hi = at(highest, (double)target_h / buckets);
    if (once) {
        lo = fmax(lo - 0.35, -1.0);
        hi = lo + 1.75;
    } else if (hi - lo < 0.75) {
        lo = fmax((lo + hi) / 2 - 0.4, -1.0);
        hi = lo + 0.75;
    }
    *low = (float)lo;
    *high = (float)hi;
}

// Wavefronts.  A lane's range holds at most 512 keys, which four wavefronts reach up to L = 8192 and eight up to 16384.  More
// than that pay where they fill an empty chip, and for long lists in long ranges, whose words are then too many for the
// registers (times of both sides; k = 32 and 5 % unless said):
//   4 or 8   L = 4608, N = 12: 101 and 153 us; 6144, N = 7: 98 and 117; 8192, N = 4, 2 %: 82 and 94; 8192, N = 2, 10 %, k = 16: 66.9
//            and 65.1; k = 128, 8192: 367 and 360; groups of 8, 8192, N = 32, 10 %: 183 and 165.  (Four have come to be better beyond
//            the line too, with lists of up to 5 %, for the mask by itself 8 %: 7000, N = 5, 5 %: 101 and 132, 8192, N = 4: 95 and 108, a
//            forward 185 and 200, at 8 % 287 and 267.)
//            Few tiles: L = 777, 294 tiles 12.1 and 11.3, 1024, 256 tiles 10.0 and 9.3, 512 11.1 and 11.6, 768, 672 tiles 13.3 and
//            16.5; 1536, 96 tiles, k = 16, 7 %: 12.2 and 12.2, 288 tiles 12.9 and 14.6; 2048, 256 tiles 12.4 and 12.0, 512 14.6
//            and 15.0; 3072, 192 tiles 16.3 and 14.7, 384 18.0 and 18.8; 4096, 512 tiles 22.1 and 21.8, 1024 32.8 and 37.9; 8192, 2 %,
//            512 29.8 and 28.0, 1024 46.8 and 50.0.
//   1 or 4   L = 128, 10 %: 1024 tiles 13.3 and 11.2, 2048 22.8 and 19.7, 4096 34.7 and 34.9.
//   2 or 4   L = 256, 10 %: 512 tiles 10.5 and 9.0, 1024 11.4 and 11.5; L = 192, 672 tiles 11.4 and 10.5, 1356 15.0 and 17.1.
inline int split_waves(const dsa_shape &sh, long long tiles)
{
    if (sh.L <= 128) return tiles <= 2048 ? 4 : 1;
    if (sh.L <= 256) return tiles <= 768 ? 4 : 2;
    if (sh.L <= 512) return 4;
    const bool four = sh.L <= 5120 || (sh.L <= 6144 && 16LL * sh.keep <= sh.L) || (sh.L <= 8192 && sh.k <= 64 && 40LL * sh.keep <= sh.L);
    if (!four) return sh.L <= 16384 ? 8 : 16;
    return tiles <= (sh.L <= 1024 ? 400 : sh.L < 2048 ? 128 : sh.L < 4096 ? 256 : sh.L / 8) ? 8 : 4;
}

// Two tiles per workgroup halve the key rows that come from L2 per unit.  They take the unit operands of both in registers, which
// only a contraction that fills its 64 slots leaves room for (k = 32 keeps two half-empty copies of each: 28 registers through
// scratch, N = 16, L = 4096, 5 % 103 -> 115 us), 16 buckets per lane instead of 32, whose bounds are worse the longer the list is,
// more wavefronts per workgroup, whose ranges may not end far beyond the head, and a grid that is not left with half a round at its end
// (waves between one and two per slot: L = 12288, N = 1, 80.6 us with one tile, 90.5 with two).  One tile and two at 1, 2, 4, 8 %:
//   rows, k = 64, N L^2 = 2^28: L = 2048 137 and 141, 144/149, 157/166, 196/213; 3072 123/126, 130/136, 151/162, 191/209; 4096 115/103,
//                126/116, 156/148, 195/194; 8192 119/93, 129/112, 162/142, 202/198; 16384 123/115, 132/133, 163/149, 240/234.  At 1 and 3 %:
//                6144 119/104, 147/139, 7168 115/110, 158/137, 10240 157/150, 182/184, 12288 140/125, 165/160; with ranges that end 2 %
//                beyond the head 5000 126/124, 155/162, 6000 118/117, 150/154, 14000 204/197, 244/244, with 14 % 4500 125/139, 150/179,
//                9000 139/156, 163/191.  Half a round is enough: L = 4096, N = 2, 24.4 and 23.3; L = 8192, N = 1, 41.4 and 38.1.
//                (These are of kernels before the bins' window and the gathered signs, which two tiles gain more from: N = 16, L = 4096, 1, 4, 6, 8, 10 % now
//                118/96, 117/107, 130/123, 137/131, 142/140; 8192, N = 4, 1 and 4 % 105/83, 129/114; 16384, N = 4, 1 % 428/372; a forward, N = 16, L = 4096, 8 %, bf16,
//                d = 128 457/445, N = 8, fp32, 6 % 312/298.  Beyond four fifths of the buckets of a lane range, 5 to 8 % from L = 5000 on, it stays at one.
//                So it does beyond 5 % with less than a round of wavefronts, whose attention in the same launch has half the workgroups, L = 4096, N = 3, 7.5 %, fp32, bf16
//                at d = 128 and at 64 89/102, 92/110 and 62.6/70.5, N = 2, 5.5 % 49.6/52.8, 49.7/53.2, 36.9/40.9 (N = 4 87.2/84.9, 91.8/88.5, 67.4/61.8), and for fp32 lists of more than
//                384 keys, whose attention does not fit the launch: 9.5 %, N = 4, 8, 16 140/145, 258/276, 509/547; 7.5 % 107/105, 210/200, 411/394.)
//   groups of 8, k = 64, N L^2 = 2^31, at 1, 2, 3, 4, 8 %: 8192 140/118, 155/138, 174/153, 185/190, 228/243; 12288 152/148, 168/165, 181/182,
//                194/195, 254/272; 16384 139/130, 153/144, 192/161, 178/223, 297/309.  A quarter of a round: 46.0 and 60.2.  (4096 146/134,
//                155/146, 166/159, 183/179, but 5000, 2 % 87/99: left at one.)
//   k = 48 rows, at 1, 2, 4 %: 4096 94/92, 101/103, 121/128; 8192 88/82, 102/96, 130/125; 16384 93/92, 104/103, 126/127; others 1 to 9 %
//                slower (10240, 1 % 120/131).  In groups never (59 registers through scratch).
inline bool split_pairs(const dsa_shape &sh, int W2, long long waves)
{
    const int NW2 = (sh.L + 128 * W2 - 1) / (128 * W2), spare = 128 * W2 * NW2 - sh.L;
    if (sh.L > 16384 || NW2 < 4 || 64 * spare > sh.L) return false;
    if (sh.vec > 1) return sh.L > 7168 && 32LL * sh.keep <= sh.L && waves >= 4096;
    if (waves < 2048 || (W2 == 16 && waves > 4096 && waves < 8192)) return false;
    if (sh.k == 48 && NW2 < 8) return false;
    const bool dense = sh.k == 64 && waves >= 4096 && (sh.dtype != DSA_F32 || sh.keep <= 384);
    return 5 * sh.keep <= 4 * 64 * W2 && sh.keep <= sh.L / (dense ? 10 : 20) + 1;
}

// Rows go over the union of their lists (tile_most, with the times) if they keep one key in so many, at least; 0: in no case.
inline int tile_part(const dsa_shape &sh, long long waves)
{
    if (sh.vec != 1 || sh.dtype != DSA_BF16 || sh.d != 64 || sh.scale == 0.f || sh.L <= 128 || waves < 2048) return 0;
    if (sh.L < 640) return 4;
    if (sh.L < 1024) return waves >= 12288 ? 10 : 8;
    if (sh.L < 2048) return waves >= 16384 ? 13 : 9;
    if (sh.L > 5120 || waves < 8192) return 12;
    return sh.L < 3000 ? 15 : sh.L < 3584 || waves < 12288 ? 16 : 20;
}

inline SplitPlan split_plan(const dsa_shape &sh, bool pairs)
{
    SplitPlan p{};
    const long long units = sh.L / sh.vec, heads = (long long)sh.B * sh.H;
    const long long tiles = heads * ((units + kTile - 1) / kTile);
    p.UT = 1;
    p.NB = 32;
    p.W = split_waves(sh, tiles);
    const int W2 = sh.L <= 8192 ? 8 : 16;
    // (where lists are dense enough for their union, for every k: the attention by itself has no use for k)
    const bool united = (long long)sh.keep * tile_part(sh, tiles * p.W) >= sh.L;
    if (pairs && !united && split_pairs(sh, W2, heads * ((units + 2 * kTile - 1) / (2 * kTile)) * W2)) {
        p.UT = 2;
        p.NB = 16;
        p.W = W2;
    }
    p.NW = (sh.L + 128 * p.W - 1) / (128 * p.W);
    const long long waves = heads * ((units + kTile * p.UT - 1) / (kTile * p.UT)) * p.W;
    split_targets(sh.L, sh.keep, p.NW, p.NB, waves <= 8192 ? 4.2 : 3.5, &p.target_l, &p.target_h);
    const double ranges = (double)sh.L / (32 * p.NW);
    split_window(p.NW == 1 ? sh.L : (int)(ranges * p.NB), !split_bins_again(sh.k, sh.vec > 1, p.NW), p.target_l, p.target_h, &p.low, &p.high);
    return p;
}

}  // namespace
}  // namespace dsa
