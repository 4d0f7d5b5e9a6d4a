// The key stream of the threshold sweep: approximate scores S~ = Q~ K~^T (paper section 3.1) of 16
// selection units (query rows, or groups of rows whose scores are summed: section 5.1) against all keys
// of their head, 16 keys at a time, from the int8 matrix cores, one wavefront on its own; plus what the
// predictor's sweeps share with it: the sum of a unit's query rows as two int8 operands and the few
// hand-written instructions that consume a score.
// Device code only; everything is internal to the translation unit that includes it.
#pragma once

#include "dsa_internal.h"
#include "wave_select.h"

namespace dsa {
namespace {

constexpr int kStreamPrefetch = 8;      // key tiles requested ahead of their use

// Geometry shared by the kernel and the host: the key range is cut into four quarters of Lq keys
// (a multiple of 32, so that a quarter is a whole number of bitmap words), quarter g = lane / 16.
__host__ __device__ inline int stream_quarter(int L) { return (L + 127) / 128 * 32; }

// sum[e] += byte e of w (signed), e = 0..3.
__device__ __forceinline__ void add_bytes(int (&sum)[4], int w)
{
#pragma unroll
    for (int e = 0; e < 4; ++e) sum[e] += (int)(int8_t)(w >> (8 * e));
}
// Four sums of up to 8 int8 values as two words of packed int8: sum = 128 * hi + lo, lo in [-64, 63].
__device__ __forceinline__ void split_sums(const int (&sum)[4], int &lo, int &hi)
{
    unsigned l = 0, h = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int top = (sum[e] + 64) >> 7;          // floor((sum + 64) / 128), |top| <= 8
        l |= ((unsigned)(sum[e] - 128 * top) & 0xffu) << (8 * e);
        h |= ((unsigned)top & 0xffu) << (8 * e);
    }
    lo = (int)l;
    hi = (int)h;
}

// Unit operands of the matrix instruction for lane (c = lane % 16, kb = lane / 16): the 16 bytes of
// the unit's query side that face part kb % (K / 16) of a key row, in the operand of the tile
// kb / (K / 16) that shares a row operand, zero in the other operands of the lane.  For VEC > 1 the
// query side is the sum of the unit's rows, split into the parts lo (qv) and hi (qh).
template <int K, int VEC>
__device__ __forceinline__ void unit_operands(const int8_t *Qunit, bool unit_live, int lane, v4i (&qv)[64 / K],
                                              v4i (&qh)[VEC == 1 ? 1 : 64 / K])
{
    constexpr int R = 64 / K, LPK = K / 16;
    const int kb = lane >> 4, sub = kb / LPK, part = kb % LPK;
    v4i lo = *reinterpret_cast<const v4i *>(Qunit + 16 * part), hi = {0, 0, 0, 0};
    if (VEC != 1) {
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            int sum[4] = {0, 0, 0, 0};
#pragma unroll
            for (int row = 0; row < VEC; ++row) add_bytes(sum, reinterpret_cast<const int *>(Qunit + row * K + 16 * part)[w]);
            int l, h;
            split_sums(sum, l, h);
            lo[w] = l;
            hi[w] = h;
        }
    }
#pragma unroll
    for (int i = 0; i < R; ++i) {
        qv[i] = (unit_live && sub == i) ? lo : v4i{0, 0, 0, 0};
        if (VEC != 1) qh[i] = (unit_live && sub == i) ? hi : v4i{0, 0, 0, 0};
    }
}

// The key stream of one wavefront: scores of tile t (16 keys x 16 units) from v_mfma_i32_16x16x64_i8.
// A matrix row is 64 bytes of contraction, i.e. R = 64 / K keys side by side: every lane loads 16
// bytes (a quarter, half or all of one key row, the widest load there is, which is what the vector
// memory path delivers best), and tile i of the R tiles that share a row operand is obtained with a
// unit operand that holds Q~ in the lanes of key i and zero in the others.  Row r of tile t is key
// (r / 4) * Lq + 4 t + r % 4, so lane (c, g) receives keys g * Lq + 4 t + {0..3} of unit c.
// Row operands sit in a ring and are requested 8 tiles before their use; the matrix core runs two
// tiles ahead of the consumer, so that the wait states between a matrix instruction and the first read
// of its result are mostly filled with work.  Whatever reads a score first must be plain code, not a
// hand-written instruction: the compiler keeps those wait states only for instructions it knows.
// Vector-wise masks (VEC = 4 or 8 query rows per unit, the group score being the sum over the rows):
// the score is linear in the query, so the unit's rows are summed first (exact in integers) and the
// sum, which needs 11 bits, is split as sum = 128 * hi + lo with lo in [-64, 63]: both parts are int8
// operands, every tile takes two matrix instructions on the same row operand, and the consumer gets
// lo_scores + 128 * hi_scores, formed two tiles after the instructions were issued.
template <int K, int VEC = 1> struct KeyStream {
    static constexpr int R = 64 / K;            // keys per matrix row = tiles per ring slot
    static constexpr int LPK = K / 16;          // lanes (16-byte parts) per key row
    static constexpr int NS = 8 / R;            // ring slots: 8 tiles in flight
    static constexpr unsigned kSlotStep = 4u * R * K;   // bytes between the rows of consecutive slots
    // tiles beyond a group's own that it touches (issues, requests): a group is plain (not SAFE) when
    // these too hold only real keys
    static constexpr int kLookahead = 2 + kStreamPrefetch;
    const int8_t *Kh;
    unsigned off0, off_last;
    v4i qv[R], qh[VEC == 1 ? 1 : R], ring[NS], p0, p1, h0, h1;     // qh, h0, h1: the hi part (VEC > 1 only)
    v4i bias;                                   // added to every score (the matrix instruction's accumulator input)

    static __device__ __forceinline__ v4i load16(const int8_t *p) { return *reinterpret_cast<const v4i *>(p); }

    template <bool SAFE> __device__ __forceinline__ void issue(int t8, int jn, unsigned next)
    {
        const int slot = (jn % 8) / R;
        p1 = __builtin_amdgcn_mfma_i32_16x16x64_i8(ring[slot], qv[jn % R], bias, 0, 0, 0);
        if (VEC != 1) h1 = __builtin_amdgcn_mfma_i32_16x16x64_i8(ring[slot], qh[jn % R], v4i{0, 0, 0, 0}, 0, 0, 0);
        if (jn % R == R - 1) {                  // the slot's last tile is on its way: request what comes 8 tiles later
            unsigned off = next + (unsigned)(jn / R) * kSlotStep;
            if (SAFE) off = min(off, off_last);
            ring[slot] = load16(Kh + off);
        }
    }
    // A group of 8 tiles starts (t8, its first tile, a multiple of 8): byte offset of the row operand
    // that holds tile t8 + 8.
    __device__ __forceinline__ unsigned begin_group(int t8) const { return off0 + (unsigned)(t8 / R + NS) * kSlotStep; }

    // Starts the stream: operands of tiles 0..7, tiles 0 and 1 issued.  Rows beyond L read row L - 1.
    // Qunit: the unit's first (or only) row of Q~; its VEC rows are contiguous.
    // Every score comes out as score + b.
    __device__ __forceinline__ void start(const int8_t *Kh_, const int8_t *Qunit, bool unit_live, int lane, int Lq, int L, int b = 0)
    {
        Kh = Kh_;
        const int r = lane & 15, kb = lane >> 4, sub = kb / LPK, part = kb % LPK;
        off0 = (unsigned)((r >> 2) * Lq + 4 * sub + (r & 3)) * (unsigned)K + 16u * part;
        off_last = (unsigned)(L - 1) * (unsigned)K + 16u * part;
        unit_operands<K, VEC>(Qunit, unit_live, lane, qv, qh);
        bias = v4i{b, b, b, b};
#pragma unroll
        for (int sl = 0; sl < NS; ++sl) ring[sl] = load16(Kh + min(off0 + (unsigned)sl * kSlotStep, off_last));
        const unsigned next = begin_group(0);
        issue<true>(0, 0, next);
        p0 = p1;
        if (VEC != 1) h0 = h1;
        issue<true>(0, 1, next);
    }
    // Scores of tile t8 + j (j = 0..7, a constant after unrolling); issues tile t8 + j + 2.
    template <bool SAFE> __device__ __forceinline__ v4i next_tile(int t8, int j, unsigned next)
    {
        v4i cur = p0;
        if (VEC != 1) cur += h0 << 7;
        p0 = p1;
        if (VEC != 1) h0 = h1;
        issue<SAFE>(t8, j + 2, next);          // tile t8 + j + 2 (for j > 5 a tile of the next group)
        return cur;
    }
};

// word = 2 * word + (v < 0) for the four scores of a tile in turn, per lane: one funnel shift each, in
// plain code, so that the compiler sees a vector instruction reading a matrix result and keeps the wait
// states that takes.  The empty statement behind them pins the shifts to their tile: without it the
// compiler gathers the shifts of a whole group of tiles behind the group's matrix instructions.
__device__ __forceinline__ void shift_in_signs(unsigned &word, v4i v)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) word = __builtin_amdgcn_alignbit(word, (unsigned)v[i], 31);
    asm volatile("" : "+v"(word));
}

// v = (key < L) ? v : INT32_MIN, per lane, as one inseparable pair (a plain compare per score of an
// unrolled round would be hoisted by the hundreds and exhaust the scalar registers).
__device__ __forceinline__ int mask_beyond(int v, int key, int L)
{
    // v may come straight from a matrix instruction, and a hand-written instruction gets no wait states
    // from the compiler: pass it through a plain vector move first (identity lane permutation)
    v = __builtin_amdgcn_update_dpp(0, v, 0xE4, 0xF, 0xF, false);
    asm("v_cmp_lt_i32 vcc, %1, %2\n\tv_cndmask_b32 %0, %3, %0, vcc" : "+v"(v) : "v"(key), "v"(L), "v"(INT32_MIN) : "vcc");
    return v;
}

// One bitmap word of a threshold sweep: 8 tiles, 32 consecutive keys of this lane's quarter, bit = score
// reaches the threshold.  The stream was started with bias = -threshold, so a score misses the
// threshold iff its sign bit is set, and one funnel shift per score moves that bit into the word.  *top: the largest of the
// 32 and what it was.
template <bool SAFE, class Stream>
__device__ __forceinline__ unsigned sweep_word(Stream &ks, int t8, int *top)
{
    const unsigned next = ks.begin_group(t8);
    unsigned word = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const v4i cur = ks.template next_tile<SAFE>(t8, j, next);
        shift_in_signs(word, cur);
        *top = max(max(cur[0], cur[1]), *top);
        *top = max(max(cur[2], cur[3]), *top);
        __builtin_amdgcn_sched_barrier(0);
    }
    return ~__brev(word);         // the first key of the word was shifted in first
}

// Largest magnitude a sweep threshold may have: score - threshold must not overflow (|score| < 2^27).
constexpr int kSweepLimit = 1 << 30;

}  // namespace
}  // namespace dsa
