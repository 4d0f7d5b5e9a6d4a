// The arithmetic of predict_split's thresholds: bins for bucket maxima, and the bracket that is swept until it is good.  Host and device.
#pragma once

#include "dsa_internal.h"

#include <math.h>

namespace dsa {
namespace {

constexpr int kBins = 128;              // histogram bins per unit

// Bin i holds the maxima from base + (i << shift) on, the last one all that lie above, too.
struct SplitBins { int base, shift; };

__host__ __device__ __forceinline__ int split_shift(unsigned range)        // range >> shift < kBins
{
    const int shift = 25 - __builtin_clz(range | 1u);
    return shift < 0 ? 0 : shift;
}
// Bins over the window of SplitPlan: reach is the distance from the smallest maximum to the mean.  (The bins are a power of two wide: what they cover
// beyond the window lies on both sides of it, where there is no second histogram three quarters of it above: clusters of
// keys put the thresholds there.)
__host__ __device__ __forceinline__ SplitBins window_bins(float mean, int least, float low, float high, bool once)
{
    const float reach = fmaxf(mean - (float)least, 0.f), range = fminf(fmaxf((high - low) * reach, 1.f), 1.0e9f);
    const int shift = split_shift((unsigned)range), base = (int)floorf(mean + low * reach) - (((kBins << shift) - (int)range) >> (once ? 2 : 1));
    return {base > least ? base : least, shift};
}
// Bins over scores from lo to hi - 1, whose last one has only what lies above.
__host__ __device__ __forceinline__ SplitBins bracket_bins(int lo, int hi)
{
    const unsigned range = (unsigned)(hi - lo);
    const int shift = split_shift(range);
    return {lo, shift + ((range + (1u << shift) - 1) >> shift >= kBins)};
}
// Below 0: the maximum lies below the bins, or the bucket is empty (the lowest number).
__host__ __device__ __forceinline__ int split_bin(SplitBins bins, int x)
{
    const int bin = __builtin_elementwise_sub_sat(x, bins.base) >> bins.shift;
    return bin < kBins - 1 ? bin : kBins - 1;
}
// Whether that many maxima between two thresholds are worth another histogram: more than twice what the targets have between them, and
// three slots of keys.  (A histogram takes a workgroup 2 to 3 us, that many keys less.  With 14 for 48: L = 4096, keep = 41, log-normal norms 80.8 and 91.3 us.)
__host__ __device__ __forceinline__ bool split_crowded(int between, int target_l, int target_h) { return between > 2 * (target_l - target_h) + 48; }
constexpr int kBinRounds = 4;           // histograms of a unit, at most

// A unit's thresholds [tl, th) and what is known about the score it looks for: it lies in [blo, bhi), and so many keys reach these.
struct SplitBracket {
    int tl, th, blo, bhi, nblo, nbhi;
    __host__ __device__ __forceinline__ bool good(int nl, int nh, int keep, int cap) const
    {
        return nh == keep || (nh < keep && nl >= keep && (nl - nh <= cap || th - tl == 1));
    }
    // After a sweep, the tries-th one, that found nl keys from tl on and nh from th on, and was not good.
    __host__ __device__ __forceinline__ void move(int nl, int nh, int keep, int cap, int tries)
    {
        const int width = th - tl;
        const bool low = nl < keep, high = nh > keep;            // the score lies below tl / at or above th
        if (low) { bhi = tl; nbhi = nl; }
        else if (high) { blo = th; nblo = nh; }
        else { blo = tl; nblo = nl; bhi = th; nbhi = nh; }
        const int span = bhi - blo, wider = 4 * (width < (1 << 24) ? width : 1 << 24);
        if (span == 1 || nblo - nbhi <= cap) {
            tl = blo;
            th = bhi;
        } else if (tries < 2 && low) {                           // just missed: a bracket of four times the width beside it
            th = bhi;
            tl = blo > th - wider ? blo : th - wider;
        } else if (tries < 2 && high) {
            tl = blo;
            th = bhi < tl + wider ? bhi : tl + wider;
        } else {                                                 // the middle third (at least one value): its bracket shrinks whatever comes out
            tl = blo + span / 3;
            th = tl + (span / 3 > 1 ? span / 3 : 1);
        }
    }
};

}  // namespace
}  // namespace dsa
