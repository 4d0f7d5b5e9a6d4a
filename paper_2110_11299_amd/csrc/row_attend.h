// Exact attention of query rows over their lists of kept keys (paper section 3.4 / 5.1), by one 64-lane wavefront: SDDMM
// (equation 2 sampled at the list), softmax over the list (equation 4) and SpMM (equation 3).  What the row kernels and the
// predictor that goes on to attend share.
//
// A key / value row of D elements is read as 16-byte pieces by LPR neighbouring lanes, so one load instruction fetches
// RPI = 64 / LPR complete, fully coalesced rows of the list.  Scores go to LDS, become weights there and never reach memory.
// Device code only; everything is internal to the translation unit that includes it.
#pragma once

#include "dsa_internal.h"
#include "wave_select.h"

#include <type_traits>

namespace dsa {
namespace {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// 16 bytes of a row: how to load them, to take a dot product of two of them and to add p times one
// of them to fp32 accumulators.
template <typename T> struct Piece;
template <> struct Piece<float> {
    static constexpr int N = 4;
    typedef float4 raw_t;
    static __device__ __forceinline__ raw_t load(const float *p) { return *reinterpret_cast<const float4 *>(p); }
    static __device__ __forceinline__ float dot(raw_t a, raw_t b)
    {
        return fmaf(a.w, b.w, fmaf(a.z, b.z, fmaf(a.y, b.y, a.x * b.x)));
    }
    // A weight as the word that is kept in LDS, what that word weighs, o += weight * b, and -a.
    static __device__ __forceinline__ unsigned weight(float p) { return __float_as_uint(p); }
    static __device__ __forceinline__ float weighs(unsigned w) { return __uint_as_float(w); }
    static __device__ __forceinline__ void axpy(float (&o)[4], unsigned w, raw_t b)
    {
        const float p = __uint_as_float(w);
        o[0] = fmaf(p, b.x, o[0]); o[1] = fmaf(p, b.y, o[1]); o[2] = fmaf(p, b.z, o[2]); o[3] = fmaf(p, b.w, o[3]);
    }
    static __device__ __forceinline__ raw_t negate(raw_t a) { return make_float4(-a.x, -a.y, -a.z, -a.w); }
};
// bfloat16: v_dot2_f32_bf16 multiplies two packed pairs and accumulates in fp32, so no element is
// ever unpacked.  For the weighted sum the weight is rounded to bfloat16 (relative 2^-8, inside the
// 2e-2 budget of bfloat16 inputs) and paired with a zero: (v0, v1) . (p, 0) = p v0, (v0, v1) . (0, p) = p v1.
template <> struct Piece<uint16_t> {
    static constexpr int N = 8;
    typedef uint4 raw_t;
    static __device__ __forceinline__ raw_t load(const uint16_t *p) { return *reinterpret_cast<const uint4 *>(p); }
    static __device__ __forceinline__ float dot2(unsigned a, unsigned b, float acc)
    {
        return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a), __builtin_bit_cast(bf16x2, b), acc, false);
    }
    static __device__ __forceinline__ float dot(raw_t a, raw_t b)
    {
        return dot2(a.w, b.w, dot2(a.z, b.z, dot2(a.y, b.y, dot2(a.x, b.x, 0.f))));
    }
    // The weight kept in LDS is the pair (p rounded to bfloat16, 0).
    static __device__ __forceinline__ unsigned weight(float p) { return __builtin_bit_cast(unsigned short, (__bf16)p); }
    static __device__ __forceinline__ float weighs(unsigned lo) { return __uint_as_float(lo << 16); }
    static __device__ __forceinline__ raw_t negate(raw_t a)
    {
        return make_uint4(a.x ^ 0x80008000u, a.y ^ 0x80008000u, a.z ^ 0x80008000u, a.w ^ 0x80008000u);
    }
    static __device__ __forceinline__ void axpy(float (&o)[8], unsigned lo, raw_t b)
    {
        const unsigned hi = lo << 16;
        o[0] = dot2(b.x, lo, o[0]); o[1] = dot2(b.x, hi, o[1]);
        o[2] = dot2(b.y, lo, o[2]); o[3] = dot2(b.y, hi, o[3]);
        o[4] = dot2(b.z, lo, o[4]); o[5] = dot2(b.z, hi, o[5]);
        o[6] = dot2(b.w, lo, o[6]); o[7] = dot2(b.w, hi, o[7]);
    }
};

// Sums of N values (1, 2 or 4) over the LPR neighbouring lanes that hold a row: a step towards fewer lanes also halves the number
// of values, so four take 10 instructions instead of 12 (LPR = 8) and their results are in one register: lane l has that of
// value piece_slot<LPR, N>(l).
template <int LPR, int N> __device__ __forceinline__ float piece_sums(const float (&a)[N], int lane)
{
    if constexpr (LPR == 1) {
        return a[0];
    } else if constexpr (N == 1) {
        const float b[1] = {halves_sum<LPR / 2>(a[0])};
        return piece_sums<LPR / 2, 1>(b, lane);
    } else {
        float b[N / 2];
#pragma unroll
        for (int i = 0; i < N / 2; ++i) b[i] = halves_sum<LPR / 2>(a[2 * i], a[2 * i + 1], lane);
        return piece_sums<LPR / 2, N / 2>(b, lane);
    }
}
template <int LPR, int N> __device__ __forceinline__ int piece_slot(int lane)
{
    if constexpr (N == 1) return 0;
    else return (lane & (LPR / 2) ? 1 : 0) + 2 * piece_slot<LPR / 2, N / 2>(lane);
}

// Sums over the 64 / LPR row groups of a wavefront, in the same way: of the E elements a lane has, it keeps the sums of the
// E * LPR / 64 from group_slot on, in o[0 ..].
template <int LPR, int E, int OFF = 32> __device__ __forceinline__ void group_sums(float (&o)[E], int lane)
{
    static_assert(LPR >= 8, "other_half<4> mixes the lanes of a group");
    if constexpr (OFF >= LPR) {
        constexpr int N = E * OFF / 64;               // that are left after this step
#pragma unroll
        for (int i = 0; i < N; ++i) o[i] = halves_sum<OFF>(o[i], o[i + N], lane);
        group_sums<LPR, E, OFF / 2>(o, lane);
    }
}
template <int LPR, int E> __device__ __forceinline__ int group_slot(int lane) { return lane / LPR * (E * LPR / kWave); }

// Geometry of a list in a wavefront: kRowGathers load instructions are in flight per row while full trips last; scores and
// weights are kept for a whole number of them.
constexpr int kRowGathers = 4;
template <typename T, int D> struct RowShape {
    static constexpr int E = Piece<T>::N, LPR = D / E, RPI = kWave / LPR, TRIP = kRowGathers * RPI, LEFT = E * LPR / kWave;
};
constexpr int kRowPad = 32;            // the longest trip

// trip(t0, TAIL): the entries [0, n) of a list.  TAIL is 0 for full trips; the last one makes TAIL gathers, those that still hold
// an entry, in code of its own for each number (under conditions they cost 2 to 5 %: SpMM, N = 16, L = 4096, keep = 205 72.8 and
// 77.3 us).
template <typename T, int D, typename F> __device__ __forceinline__ void row_trips(int n, F &&trip)
{
    constexpr int RPI = RowShape<T, D>::RPI, TRIP = RowShape<T, D>::TRIP;
    int t0 = 0;
    for (; t0 + TRIP <= n; t0 += TRIP) trip(t0, std::integral_constant<int, 0>{});
    const int rest = n - t0;
    if (rest > 3 * RPI) trip(t0, std::integral_constant<int, 4>{});
    else if (rest > 2 * RPI) trip(t0, std::integral_constant<int, 3>{});
    else if (rest > RPI) trip(t0, std::integral_constant<int, 2>{});
    else if (rest > 0) trip(t0, std::integral_constant<int, 1>{});
}

// Gathers of one trip: row at(r, t) of every list, entries beyond the list as its last one.
template <typename T, int D, int NR, int TAIL, typename At>
__device__ __forceinline__ void row_gather(typename Piece<T>::raw_t (&x)[NR][kRowGathers], const T *head, At &&at, int t0, int n, int lane)
{
    typedef RowShape<T, D> G;
    const unsigned piece_at = lane % G::LPR * 16u;
#pragma unroll
    for (int u = 0; u < kRowGathers; ++u) {
        if (TAIL && u >= TAIL) continue;
        const int t = t0 + u * G::RPI + lane / G::LPR;
#pragma unroll
        for (int r = 0; r < NR; ++r)
            x[r][u] = Piece<T>::load(reinterpret_cast<const T *>(reinterpret_cast<const char *>(head) +
                                                                 (size_t)(at(r, TAIL ? min(t, n - 1) : t) + piece_at)));
    }
}

// q . k of the first n entries of NR lists to sc[r * pad + t], and something to entries behind them, up to the end of the last trip at
// most.  at(r, t): byte offset of the key row of entry t inside the head.  m[r]: this lane's share of the maximum.
template <typename T, int D, int NR, typename At>
__device__ __forceinline__ void row_scores(const T *Kh, const typename Piece<T>::raw_t (&q)[NR], At &&at, float *sc, int pad, int n,
                                           int lane, float (&m)[NR])
{
    typedef RowShape<T, D> G;
#pragma unroll
    for (int r = 0; r < NR; ++r) m[r] = -INFINITY;
    row_trips<T, D>(n, [&](int t0, auto tail) {
        constexpr int TAIL = decltype(tail)::value, NS = NR == 1 && (TAIL == 1 || TAIL == 2) ? TAIL : kRowGathers;     // sums that are taken
        typename Piece<T>::raw_t kv[NR][kRowGathers];
        if (TAIL) {
#pragma unroll
            for (int r = 0; r < NR; ++r)
#pragma unroll
                for (int u = TAIL; u < NS; ++u) kv[r][u] = q[r];
        }
        row_gather<T, D, NR, TAIL>(kv, Kh, at, t0, n, lane);
        // One row of d = 128 at a time: whole sums for every gather.  The merged ones take fewer instructions, but where few rows with
        // long lists leave a SIMD four wavefronts their chain is waited for: SDDMM, bf16, N = 1, L = 4096, 800 keys 34.6 and 31.0 us,
        // attention 56.8 and 52.7, fp32, 500 keys 36.7 and 35.0; N = 4, L = 16384, 164 keys 102 and 102; CSR lists up to 2 % slower.
        if constexpr (NR == 1 && D == 128 && TAIL == 0) {
            float s[kRowGathers];
#pragma unroll
            for (int u = 0; u < kRowGathers; ++u) {
                const float part[1] = {Piece<T>::dot(q[0], kv[0][u])};
                s[u] = piece_sums<G::LPR, 1>(part, lane);
            }
#pragma unroll
            for (int u = 0; u < kRowGathers; ++u) {
                m[0] = fmaxf(m[0], s[u]);
                sc[t0 + u * G::RPI + lane / G::LPR] = s[u];          // every lane of the group writes the same value
            }
            return;
        }
        const int t = t0 + piece_slot<G::LPR, NS>(lane) * G::RPI + lane / G::LPR;
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            float part[NS];
#pragma unroll
            for (int u = 0; u < NS; ++u) part[u] = Piece<T>::dot(q[r], kv[r][u]);
            const float s = piece_sums<G::LPR, NS>(part, lane);
            if (!TAIL || t < n) m[r] = fmaxf(m[r], s);
            sc[r * pad + t] = s;                      // lanes with the same entry write the same value
        }
    });
}

// o[r] += weight * value row over the entries of this lane group.  sw: the weights; entries beyond n weigh 0, and their values are 0 in
// fp32, since 0 times an infinite value would not be.  (In bf16 an infinite value makes NaN of the neighbouring column anyway, whose
// product with the weight's zero is NaN.)
template <typename T, int D, int NR, typename At>
__device__ __forceinline__ void row_values(const T *Vh, At &&at, const unsigned *sw, int pad, int n, int lane,
                                           float (&o)[NR][Piece<T>::N])
{
    typedef RowShape<T, D> G;
    row_trips<T, D>(n, [&](int t0, auto tail) {
        constexpr int TAIL = decltype(tail)::value;
        typename Piece<T>::raw_t vv[NR][kRowGathers];
        row_gather<T, D, NR, TAIL>(vv, Vh, at, t0, n, lane);
        if constexpr (TAIL != 0 && sizeof(T) == 4) {
            const bool in = t0 + (TAIL - 1) * G::RPI + lane / G::LPR < n;
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                typename Piece<T>::raw_t &x = vv[r][TAIL - 1];
                x.x = in ? x.x : 0;
                x.y = in ? x.y : 0;
                x.z = in ? x.z : 0;
                x.w = in ? x.w : 0;
            }
        }
        unsigned w[NR][kRowGathers];
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
            for (int u = 0; u < kRowGathers; ++u) w[r][u] = sw[r * pad + t0 + u * G::RPI + lane / G::LPR];
#pragma unroll
        for (int u = 0; u < kRowGathers; ++u) {
            if (TAIL && u >= TAIL) continue;      // (0 times an infinite value would not be 0)
#pragma unroll
            for (int r = 0; r < NR; ++r) Piece<T>::axpy(o[r], w[r][u], vv[r][u]);
        }
    });
}

// Scores in LDS become weights exp(factor * (score - m)), 0 in [n, pad).  ROUNDED: z gets the sum of what the products will use
// instead of the fp32 weights.
template <typename T, int NR, bool ROUNDED>
__device__ __forceinline__ void row_weights(unsigned *sw, int pad, int n, float factor, const float (&m)[NR], int lane, float (&z)[NR])
{
    for (int t = lane; t < pad; t += kWave) {
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const float p = t < n ? __expf(factor * (__uint_as_float(sw[r * pad + t]) - m[r])) : 0.f;
            const unsigned w = Piece<T>::weight(p);
            z[r] += ROUNDED ? Piece<T>::weighs(w) : p;
            sw[r * pad + t] = w;
        }
    }
}

// This lane's sums over all groups, times inv, to the row `out` of O.
template <typename T, int D>
__device__ __forceinline__ void row_store(float *out, float (&o)[Piece<T>::N], float inv, int lane)
{
    typedef RowShape<T, D> G;
    group_sums<G::LPR, G::E>(o, lane);
    float *dst = out + lane % G::LPR * G::E + group_slot<G::LPR, G::E>(lane);
    if (G::LEFT == 2) *reinterpret_cast<float2 *>(dst) = make_float2(o[0] * inv, o[1] * inv);
    else dst[0] = o[0] * inv;
}

// NR rows with lists of the same length, from scores to O: q are their pieces, out[r] their rows of O, lds room for
// NR * pad words (pad: n rounded up to kRowPad) of this wavefront's own.
template <typename T, int D, int NR, typename At>
__device__ __forceinline__ void attend_rows(const T *Kh, const T *Vh, typename Piece<T>::raw_t (&q)[NR], At &&at, unsigned *lds, int pad, int n,
                                            float scale, float *const (&out)[NR], int lane)
{
    // the scores are kept as sign(scale) * q.k and the factor |scale| waits for the exponential
    if (scale < 0.f) {
#pragma unroll
        for (int r = 0; r < NR; ++r) q[r] = Piece<T>::negate(q[r]);
    }
    float m[NR], z[NR], o[NR][Piece<T>::N];
    row_scores<T, D, NR>(Kh, q, at, reinterpret_cast<float *>(lds), pad, n, lane, m);
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        m[r] = wave_all_max(m[r]);
        z[r] = 0.f;
#pragma unroll
        for (int e = 0; e < Piece<T>::N; ++e) o[r][e] = 0.f;
    }
    wave_lds_sync();
    row_weights<T, NR, true>(lds, pad, n, fabsf(scale), m, lane, z);
    wave_lds_sync();
    row_values<T, D, NR>(Vh, at, lds, pad, n, lane, o);
    wave_lds_sync();                                   // the next rows overwrite the weights
#pragma unroll
    for (int r = 0; r < NR; ++r) row_store<T, D>(out[r], o[r], 1.f / wave_all_sum(z[r]), lane);
}

// What a workgroup attends with.
struct AttendArgs {
    const void *Q, *K, *V;
    float *O;
    float scale;
    int d, pad;                         // list length rounded up to kRowPad
    int most;                           // tile_attend.h: keys of the longest union
    unsigned lds;                       // and bytes of LDS
};

// Rows a wavefront attends to at a time: a gather of each is as good as another gather of one, and the steps between the gathers
// overlap.  bf16 1, 2, 4 rows, k = 32: N = 16, L = 4096, keep = 205 211.7, 202.2, 210.4 us, keep = 410 323, 307, 356; fp32 (a
// quarter of the sums per row) 2 and 4, k = 16: N = 512, L = 256, keep = 26 113.7 and 103.8, N = 128, L = 1024, keep = 102 256 and 249.
template <typename T> constexpr int attend_rows_at_once() { return sizeof(T) == 2 ? 2 : 4; }

// The rows of the workgroup's nu units, by `waves` of its wavefronts (at most all).  image: the units' lists; lds: room for
// attend_rows_at_once() * pad words for each of them.
template <typename T, int D>
__device__ __forceinline__ void attend_block(const AttendArgs &a, const uint16_t *image, unsigned *lds, int L, int keep, int vec, unsigned n, int u0, int nu,
                                             int waves)
{
    const int lane = threadIdx.x & (kWave - 1), wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), W = min(waves, (int)(blockDim.x / kWave));
    if (wv >= W) return;
    constexpr int NR = attend_rows_at_once<T>(), LPR = RowShape<T, D>::LPR, E = Piece<T>::N;
    const size_t head = (size_t)n * L * D;
    const T *Kh = static_cast<const T *>(a.K) + head, *Vh = static_cast<const T *>(a.V) + head, *Qh = static_cast<const T *>(a.Q) + head;
    lds += wv * NR * a.pad;
    const int total = nu * vec;
    for (int p = wv; NR * p < total; p += W) {
        typename Piece<T>::raw_t q[NR];
        const uint16_t *list[NR];
        float *out[NR];
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int j = min(NR * p + r, total - 1);          // (a row that is there twice is written twice)
            const size_t row = (size_t)(u0 * vec + j) * D;
            q[r] = Piece<T>::load(Qh + row + lane % LPR * E);
            list[r] = image + (vec == 1 ? j : j / vec) * keep;
            out[r] = a.O + head + row;
        }
        auto at = [&](int r, int t) { return (unsigned)list[r][t] * (unsigned)(D * sizeof(T)); };
        attend_rows<T, D, NR>(Kh, Vh, q, at, lds, a.pad, keep, a.scale, out, lane);
    }
}

}  // namespace
}  // namespace dsa
