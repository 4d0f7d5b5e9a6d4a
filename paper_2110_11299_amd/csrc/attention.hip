// Exact attention at the kept positions (paper section 3.4 / 5.1): SDDMM (equation 2 sampled at
// the mask), softmax over the kept entries (equation 4) and SpMM (equation 3).
//
// Row kernel.  One 64-lane wavefront owns one query row, with the loops of row_attend.h.  The kernel is bound by the gathers
// (about 1 flop per byte), so everything else stays on chip: S and P never reach HBM in the fused mode.
#include "dsa_internal.h"
#include "attention_api.h"
#include "predict_api.h"
#include "tile_attend.h"

#include <algorithm>

namespace dsa {
namespace {

constexpr int kRowWaves = 4;          // query rows (wavefronts) per workgroup
constexpr int kMaxKeep = 4096;        // list and scores of a row in LDS: 4 waves * 4096 * 8 B = 128 KB

// The unit that row i of head n belongs to; vec is 1, 4 or 8.  (Two divisions were 60 of the 330 instructions of a row of 3 keys.)
__device__ __forceinline__ size_t unit_of(unsigned n, unsigned i, int L, int vec)
{
    const int shift = __builtin_ctz(vec);
    return (size_t)n * (L >> shift) + (i >> shift);
}

// MODE kFused: Q,K,V,idx -> O.  kSddmm: Q,K,idx -> S.  kSpmm: Pin,V,idx -> O.
template <typename T, int D, int MODE>
__global__ __launch_bounds__(kRowWaves *kWave) void attention_rows(
    const T *__restrict__ Q, const T *__restrict__ K, const T *__restrict__ V,
    const int32_t *__restrict__ idx, const float *__restrict__ Pin, float *__restrict__ S,
    float *__restrict__ O, int L, int keep, int keep_pad, int vec, float scale, unsigned total_rows)
{
    typedef Piece<T> P;
    typedef typename P::raw_t raw_t;
    constexpr int E = P::N;               // elements per lane
    extern __shared__ unsigned lds_words[];

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int sub = lane % RowShape<T, D>::LPR;
    const unsigned vblock = xcd_contiguous(blockIdx.x, gridDim.x);
    const unsigned row = vblock * kRowWaves + wave;                 // wavefront-uniform from here on
    if (row >= total_rows) return;                        // the whole wavefront: nothing below is shared
    const unsigned n = row / (unsigned)L, i = row % (unsigned)L;
    const int32_t *list = idx + unit_of(n, i, L, vec) * keep;
    // per wavefront in LDS: the row's key list, as the byte offset of every key row inside its head
    // (keys clamped into [0, L), so that no idx can send a gather outside K / V), filled up with its last key, and its scores,
    // later (or from the start, when the weights are given) its weights
    constexpr unsigned kRowBytes = D * sizeof(T);
    unsigned *sl = lds_words + wave * 2 * keep_pad, *sw = sl + keep_pad;
    for (int t = lane; t < keep_pad; t += kWave) sl[t] = (unsigned)min(max(list[min(t, keep - 1)], 0), L - 1) * kRowBytes;
    auto at = [&](int, int t) { return sl[t]; };
    const T *Kh = K + (size_t)n * L * D, *Vh = V + (size_t)n * L * D;
    raw_t q[1];
    if (MODE != kSpmm) q[0] = P::load(Q + (size_t)row * D + sub * E);
    wave_lds_sync();
    if (MODE == kFused) {
        attend_rows<T, D, 1>(Kh, Vh, q, at, sw, keep_pad, keep, scale, {O + (size_t)row * D}, lane);
    } else if (MODE == kSddmm) {
        float m[1];
        float *sc = reinterpret_cast<float *>(sw);
        row_scores<T, D, 1>(Kh, q, at, sc, 0, keep, lane, m);
        // the row of scores leaves in one piece: consecutive lanes, consecutive entries
        wave_lds_sync();
        for (int t = lane; t < keep; t += kWave) S[(size_t)row * keep + t] = sc[t] * scale;
    } else {
        // the given weights come in the same way and wait in LDS in the form the products take them
        for (int t = lane; t < keep_pad; t += kWave) sw[t] = t < keep ? P::weight(Pin[(size_t)row * keep + t]) : 0u;
        wave_lds_sync();
        float o[1][E];
#pragma unroll
        for (int e = 0; e < E; ++e) o[0][e] = 0.f;
        row_values<T, D, 1>(Vh, at, sw, 0, keep, lane, o);
        row_store<T, D>(O + (size_t)row * D, o[0], 1.f, lane);
    }
}

// Row kernel for masks in CSR form (threshold masks, section 3.1: the count per row varies).  Same
// wavefront-per-row scheme and the same gather loops as attention_rows, fused only; a row's list is taken in chunks of
// kCsrChunk keys with a running maximum, so that any count fits the same LDS: when a later chunk
// raises the maximum, the sums so far are rescaled by exp(m_old - m_new).  4 KB of LDS per row leave room for eight rows
// per SIMD, and most lists are one chunk.  N = 16, L = 2048, about 102 keys a row: 91 -> 54 us against tests per key,
// a conversion per weight and gather, and 8 KB per row.
// WAVES: rows of a workgroup.  With four, their places wait for the longest of four lists, with one, neighbours that share a list do not
// share an L1.  One and four (the kernel alone): single rows, fp32, N = 77, L = 2056, 27 keys a row (standard deviation 42) 105.9 and
// 117.7 us, bf16, N = 16, L = 2048, 109 (95) 42.4 and 43.9; groups of 4, bf16, d = 128, N = 148, L = 520, 23 (23) 49.8 and 51.5, but fp32,
// N = 44, L = 1048, 27 (31) 61.6 and 60.5; groups of 8, fp32, N = 15, L = 5032, 145 (180) 251.5 and 237.2, bf16, N = 124, L = 1296, 103 (81)
// 170.3 and 167.4, but d = 128, N = 21, L = 2336, 36 (50) 51.2 and 52.2.  Groups of 8 take four (their rows are a multiple of it).
// The weights are summed in fp32 as they are made; only the products take them rounded, if T is bfloat16.
constexpr int kCsrChunk = 512;
static_assert(kCsrChunk % kRowPad == 0, "a full chunk needs no padding");

template <typename T, int D, int WAVES>
__global__ __launch_bounds__(WAVES *kWave) void attention_rows_csr(
    const T *__restrict__ Q, const T *__restrict__ K, const T *__restrict__ V,
    const int32_t *__restrict__ row_ptr, const int32_t *__restrict__ col, float *__restrict__ O, int L, int vec, float scale)
{
    typedef Piece<T> P;
    constexpr int E = P::N;
    constexpr unsigned kRowBytes = D * sizeof(T);
    __shared__ unsigned lists[WAVES][kCsrChunk], weights[WAVES][kCsrChunk];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int sub = lane % RowShape<T, D>::LPR;
    unsigned *sl = lists[wave], *sw = weights[wave];       // the list; scores, then weights
    const unsigned row = xcd_contiguous(blockIdx.x, gridDim.x) * WAVES + wave;
    const unsigned n = row / (unsigned)L, i = row % (unsigned)L;
    const size_t u = unit_of(n, i, L, vec);
    const int beg = row_ptr[u];
    const int cnt = max(row_ptr[u + 1] - beg, 0);
    // the scores are kept as sign(scale) * q.k and the factor |scale| waits for the exponential
    typename P::raw_t q[1] = {P::load(Q + (size_t)row * D + sub * E)};
    if (scale < 0.f) q[0] = P::negate(q[0]);
    const float factor = fabsf(scale);
    const T *Kh = K + (size_t)n * L * D, *Vh = V + (size_t)n * L * D;
    auto at = [&](int, int t) { return sl[t]; };

    float m[1] = {-INFINITY}, z[1] = {0.f}, o[1][E];
#pragma unroll
    for (int e = 0; e < E; ++e) o[0][e] = 0.f;
    for (int c0 = 0; c0 < cnt; c0 += kCsrChunk) {
        const int nk = min(kCsrChunk, cnt - c0), pad = (nk + kRowPad - 1) / kRowPad * kRowPad;
        const int32_t *list = col + beg + c0;
        for (int t = lane; t < pad; t += kWave) sl[t] = (unsigned)min(max(list[min(t, nk - 1)], 0), L - 1) * kRowBytes;
        wave_lds_sync();
        float m_new[1];
        row_scores<T, D, 1>(Kh, q, at, reinterpret_cast<float *>(sw), 0, nk, lane, m_new);
        m_new[0] = fmaxf(m[0], wave_all_max(m_new[0]));
        if (c0 > 0) {
            const float f = __expf(factor * (m[0] - m_new[0]));
            z[0] *= f;
#pragma unroll
            for (int e = 0; e < E; ++e) o[0][e] *= f;
        }
        m[0] = m_new[0];
        wave_lds_sync();
        row_weights<T, 1, false>(sw, pad, nk, factor, m, lane, z);
        wave_lds_sync();
        row_values<T, D, 1>(Vh, at, sw, 0, nk, lane, o);
        wave_lds_sync();                                   // the next chunk overwrites list and weights
    }
    // a row without keys (not made by the predictor) gives 0
    row_store<T, D>(O + (size_t)row * D, o[0], cnt > 0 ? 1.f / wave_all_sum(z[0]) : 0.f, lane);
}

// Measurement aid: the gathers of attention_rows and nothing else.  Same launch shape, same key list
// staged in LDS, same 16-byte pieces with four gathers in flight per lane, first over K and then over V;
// the pieces are only folded into one word per row so that the loads cannot be dropped.  Its rate, in
// gathered bytes per second, is the roof the memory hierarchy (L1 / L2, where K and V of a head live)
// sets for this access pattern: the yardstick for attention_rows.
template <typename T, int D>
__global__ __launch_bounds__(kRowWaves *kWave) void gather_probe(const T *__restrict__ K, const T *__restrict__ V,
                                                                 const int32_t *__restrict__ idx,
                                                                 unsigned *__restrict__ sink, int L, int keep,
                                                                 int keep_pad, int vec, unsigned total_rows)
{
    typedef Piece<T> P;
    constexpr unsigned kRowBytes = D * sizeof(T);
    extern __shared__ float lds_scores[];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const unsigned row = xcd_contiguous(blockIdx.x, gridDim.x) * kRowWaves + wave;
    const bool live = row < total_rows;
    const unsigned r = live ? row : total_rows - 1;
    const unsigned n = r / (unsigned)L, i = r % (unsigned)L;
    const int32_t *list = idx + unit_of(n, i, L, vec) * keep;
    // the same padded list of byte offsets as in attention_rows, the same address arithmetic
    unsigned *sl = reinterpret_cast<unsigned *>(lds_scores) + wave * keep_pad;
    for (int t = lane; t < keep_pad; t += kWave) sl[t] = (unsigned)min(max(list[min(t, keep - 1)], 0), L - 1) * kRowBytes;
    wave_lds_sync();
    unsigned acc = 0;
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
        const T *Xh = (pass ? V : K) + (size_t)n * L * D;
        row_trips<T, D>(keep, [&](int t0, auto tail) {
            typename P::raw_t x[1][kRowGathers];
            if (decltype(tail)::value) {
#pragma unroll
                for (int u = decltype(tail)::value; u < kRowGathers; ++u) x[0][u] = typename P::raw_t{};
            }
            row_gather<T, D, 1, decltype(tail)::value>(x, Xh, [&](int, int t) { return sl[t]; }, t0, keep, lane);
#pragma unroll
            for (int u = 0; u < kRowGathers; ++u) {
                const uint4 w = __builtin_bit_cast(uint4, x[0][u]);
                acc ^= (w.x ^ w.y) ^ (w.z ^ w.w);
            }
        });
    }
    if (live) sink[(size_t)r * kWave + lane] = acc;
}

// Group kernel for the staged entry points (SDDMM, SpMM) of the vector-wise mask with bfloat16 inputs.  The 8 query rows of
// a group share one key list, so each gathered key / value row serves 8 rows and the products become small dense
// contractions for the bf16 matrix cores (v_mfma_f32_16x16x32_bf16, fp32 accumulate).  One wavefront owns one group.
//   Scores: the gathered key rows are the A operand (16 keys per tile: lane (r = lane%16, g = lane/16) holds key r,
//   elements [8g, 8g+8) of each 32-element step), the 8 query rows (padded to 16) the B operand.  Lane (c, g) then owns,
//   for query c, keys 4g..4g+3 of the tile.  Scaled scores go to LDS and leave as whole rows.
//   Output: over a 32-key step lane group g owns keys {4g+i} of the first tile and {16+4g+i} of the second: the weights of
//   these 8, rounded to bfloat16 (relative 2^-8, inside the 2e-2 budget), are the A operand (query c, slots of g).  The
//   32 gathered value rows go through LDS once and come back transposed (ds_read_tr16_b64) as the B operand with the same
//   slot order (lane (c, g): column c of the rows that are g's slots).
constexpr int kGroupWaves = 4;


// (The launch bound is twice the launched size: with at most 256 registers per lane the compiler
// gives the matrix core plain VGPR destinations instead of accumulation registers that every
// other instruction would have to copy from.)
// MODE kSddmm: Q,K,idx -> S (scaled scores of the 8 rows).  kSpmm: Pin,V,idx -> O.
template <int D, int MODE>
__global__ __launch_bounds__(2 * kGroupWaves *kWave) void attention_groups_bf16(
    const uint16_t *__restrict__ Q, const uint16_t *__restrict__ K, const uint16_t *__restrict__ V,
    const int32_t *__restrict__ idx, const float *__restrict__ Pin, float *__restrict__ S, float *__restrict__ O,
    int L, int keep, int keep_pad, float scale, unsigned total_groups)
{
    constexpr int KS = D / 32;             // contraction steps of Q K^T
    constexpr int CT = D / 16;             // 16-column tiles of the output
    constexpr int VROW = D * 2 + 16;       // bytes of one value row in LDS (padded against bank conflicts)
    constexpr int LPR = D / 8;             // lanes that load one row as 16-byte pieces
    constexpr int RPI = kWave / LPR;       // rows per load instruction
    extern __shared__ __attribute__((aligned(16))) char lds_raw[];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int c = lane & 15, g = lane >> 4;
    const size_t per_wave = (size_t)9 * keep_pad * sizeof(float) + 32 * VROW;
    float *sS = reinterpret_cast<float *>(lds_raw + wave * per_wave);          // [8][keep_pad]
    int *sl = reinterpret_cast<int *>(sS + 8 * keep_pad);                      // [keep_pad] key list
    char *sV = reinterpret_cast<char *>(sl + keep_pad);                        // [32][VROW]

    const unsigned vblock = xcd_contiguous(blockIdx.x, gridDim.x);
    const unsigned grp = vblock * kGroupWaves + wave;
    const bool live = grp < total_groups;
    const unsigned gi = live ? grp : total_groups - 1;     // dead waves shadow a real group, write nothing
    const unsigned G = L / 8, n = gi / G, u = gi % G;
    const int32_t *list = idx + (size_t)gi * keep;
    const uint16_t *Kh = K + (size_t)n * L * D, *Vh = V + (size_t)n * L * D;

    bf16x8 qop[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const uint4 raw = (MODE != kSpmm && c < 8) ? *reinterpret_cast<const uint4 *>(Q + ((size_t)n * L + u * 8 + c) * D + 32 * s + 8 * g)
                                : make_uint4(0, 0, 0, 0);
        qop[s] = __builtin_bit_cast(bf16x8, raw);
    }

    // the group's key list once into LDS, clamped into [0, L) (no idx can send a gather outside K / V)
    // and padded with its last entry
    for (int t = lane; t < keep_pad; t += kWave) sl[t] = min(max(list[min(t, keep - 1)], 0), L - 1);
    wave_lds_sync();

    // scores of all kept keys -> LDS.  The key rows of a step (32 keys) are gathered the way the value rows are below:
    // D / 8 neighbouring lanes fetch one row as 16-byte pieces (whole cache lines per row, which is what the vector memory
    // path serves best; fetched straight into the operand layout, 16 lanes take 16 bytes of 16 different rows each and the
    // same bytes come at a third of the rate), pass through the value tile's LDS and come back as the first operand of
    // the matrix instruction.  The rows of step t + 1 are requested before step t is consumed.
    constexpr int VP = 32 / RPI;           // load instructions per step of 32 rows
    const int vrow = lane / LPR, vpiece = lane % LPR;
    if (MODE == kSddmm) {
        v4u kring[VP];
#pragma unroll
        for (int rr = 0; rr < VP; ++rr)
            kring[rr] = *reinterpret_cast<const v4u *>(Kh + (size_t)sl[rr * RPI + vrow] * D + vpiece * 8);
        for (int t0 = 0; t0 < keep_pad; t0 += 32) {
#pragma unroll
            for (int rr = 0; rr < VP; ++rr) *reinterpret_cast<v4u *>(sV + (rr * RPI + vrow) * VROW + vpiece * 16) = kring[rr];
            const int tn = min(t0 + 32, keep_pad - 32);
#pragma unroll
            for (int rr = 0; rr < VP; ++rr)
                kring[rr] = *reinterpret_cast<const v4u *>(Kh + (size_t)sl[tn + rr * RPI + vrow] * D + vpiece * 8);
            wave_lds_sync();
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const int tile = t0 + 16 * half;
                v4f acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    const bf16x8 ka = *reinterpret_cast<const bf16x8 *>(sV + (16 * half + c) * VROW + (32 * s + 8 * g) * 2);
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka, qop[s], acc, 0, 0, 0);
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[i] *= scale;
                if (c < 8) *reinterpret_cast<v4f *>(sS + c * keep_pad + tile + 4 * g) = acc;
            }
            wave_lds_sync();       // the next step overwrites the tile
        }
        // the 8 rows of scores leave through LDS: consecutive lanes write consecutive entries of a row
        if (live) {
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                float *dst = S + ((size_t)n * L + u * 8 + r) * keep;
                for (int t = lane; t < keep; t += kWave) dst[t] = sS[r * keep_pad + t];
            }
        }
        return;
    }
    // the given weights come in the same way (0 beyond the list)
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const float *src = Pin + ((size_t)n * L + u * 8 + r) * keep;
        for (int t = lane; t < keep_pad; t += kWave) sS[r * keep_pad + t] = t < keep ? src[t] : 0.f;
    }
    wave_lds_sync();

    v4f o[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) o[ct] = v4f{0.f, 0.f, 0.f, 0.f};
    const float *srow = sS + (c & 7) * keep_pad + 4 * g;
    const char *block = sV + (4 * g + (c >> 2)) * VROW + 8 * (c & 3);      // what a lane contributes to a transposing read
    v4u vring[VP];
#pragma unroll
    for (int rr = 0; rr < VP; ++rr) vring[rr] = *reinterpret_cast<const v4u *>(Vh + (size_t)sl[rr * RPI + vrow] * D + vpiece * 8);
    for (int t0 = 0; t0 < keep_pad; t0 += 32) {
        // 32 gathered value rows -> LDS, and the request for the rows of the next step
#pragma unroll
        for (int rr = 0; rr < VP; ++rr) *reinterpret_cast<v4u *>(sV + (rr * RPI + vrow) * VROW + vpiece * 16) = vring[rr];
        const int tn = min(t0 + 32, keep_pad - 32);
#pragma unroll
        for (int rr = 0; rr < VP; ++rr)
            vring[rr] = *reinterpret_cast<const v4u *>(Vh + (size_t)sl[tn + rr * RPI + vrow] * D + vpiece * 8);
        // weights of this lane's 8 slots
        const v4f s0 = *reinterpret_cast<const v4f *>(srow + t0);
        const v4f s1 = *reinterpret_cast<const v4f *>(srow + t0 + 16);
        bf16x8 pa;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            pa[i] = (__bf16)s0[i];
            pa[4 + i] = (__bf16)s1[i];
        }
        wave_lds_sync();
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            union { s16x4 half[2]; bf16x8 all; } vb;
            vb.half[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(block + 32 * ct));
            vb.half[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(block + 16 * VROW + 32 * ct));
            o[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pa, vb.all, o[ct], 0, 0, 0);
        }
        wave_lds_sync();       // the next step overwrites the value tile
    }
    // lane (c, g) holds O[query 4g+i][16 ct + c]
    if (live && g < 2) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float *out = O + ((size_t)n * L + u * 8 + 4 * g + i) * D + c;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) out[16 * ct] = o[ct][i];
        }
    }
}

template <int D, int VEC>
__global__ __launch_bounds__(kGroupWaves *kWave, 4) void attention_units_bf16(
    const uint16_t *__restrict__ Q, const uint16_t *__restrict__ K, const uint16_t *__restrict__ V,
    const int32_t *__restrict__ idx, float *__restrict__ O, int L, int keep, int keep_pad, float scale, unsigned total_units)
{
    extern __shared__ __attribute__((aligned(16))) char lds_raw[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    char *tile = lds_raw + wave * (unit_tile_bytes<D>() + keep_pad * 4);
    const unsigned unit = xcd_contiguous(blockIdx.x, gridDim.x) * kGroupWaves + wave;
    if (unit >= total_units) return;       // the whole wavefront: nothing below is shared
    const unsigned G = L / VEC, n = unit / G, u = unit % G;
    const int32_t *list = idx + (size_t)unit * keep;
    const size_t head = (size_t)n * L * D, first = head + (size_t)u * VEC * D;
    attend_unit<D, true>(Q + first, K + head, V + head, [&](int t) { return min(max(list[t], 0), L - 1); }, O + first, VEC, keep, keep_pad, scale, tile);
}

// Fine-grained rows in bfloat16, 16 to a workgroup, over the union of their lists (tile_attend.h): what predict_split does with lists that
// it has made, for lists that are given.  The union comes from a word of LDS per two keys (which needs their 2 L bytes to fit what the
// tiles take later).  Rows that have a key twice, as entries outside of [0, L) may when they are clamped, and sums that are not
// finite go to the loops of attention_rows.
__global__ __launch_bounds__(512, 4) void attention_tiles_bf16(AttendArgs a, const int32_t *__restrict__ idx, int L, int keep, int tiles_per_head)
{
    extern __shared__ __align__(16) char lds_raw[];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = __builtin_amdgcn_readfirstlane(tid / kWave), T = blockDim.x, W = T / kWave;
    const unsigned wg = xcd_contiguous(blockIdx.x, gridDim.x), n = wg / (unsigned)tiles_per_head;
    const int u0 = (int)(wg % (unsigned)tiles_per_head) * kTileRows, nu = min(kTileRows, L - u0);
    char *room = lds_raw;
    const TileLds at(W, a.most);
    unsigned *masks = reinterpret_cast<unsigned *>(room + at.work), *entries = reinterpret_cast<unsigned *>(room + at.list);
    const int words = (L + 1) / 2;
    for (int e = tid; 4 * e < words; e += T) reinterpret_cast<v4u *>(masks)[e] = v4u{0, 0, 0, 0};
    const int32_t *lists = idx + ((size_t)n * L + u0) * keep;
    __syncthreads();
    for (int e = tid, r = tid / keep, t = tid % keep; e < nu * keep; e += T) {      // entry t of row r
        const unsigned key = min(max(lists[e], 0), L - 1);
        atomicOr(&masks[key >> 1], 1u << (r + 16 * (key & 1)));
        r += T / keep;
        t += T % keep;
        if (t >= keep) {
            t -= keep;
            ++r;
        }
    }
    __syncthreads();
    const int share = (words + T - 1) / T * kWave, first = wv * share;          // words of a wavefront
    int mine = 0, kept = 0;
    for (int e = first + lane; e - lane < first + share; e += kWave) {
        const unsigned m = e < words ? masks[e] : 0u;
        mine += __popcll(__ballot((m & 0xffffu) != 0)) + __popcll(__ballot((m >> 16) != 0));
        kept += __popc(m);
    }
    kept = wave_sum(kept);
    int *counts = reinterpret_cast<int *>(room);
    if (lane == 0) {
        counts[2 * wv] = mine;
        counts[2 * wv + 1] = kept;
    }
    __syncthreads();
    int total = 0, pos = 0, all = 0;
    for (int w = 0; w < W; ++w) {
        pos += w < wv ? counts[2 * w] : 0;
        total += counts[2 * w];
        all += counts[2 * w + 1];
    }
    total = __builtin_amdgcn_readfirstlane(total);
    if (__builtin_amdgcn_readfirstlane(all) == nu * keep) {
        if (wv == 0) tile_fill(entries, total, lane);
        for (int e = first + lane; e - lane < first + share; e += kWave) {
            const unsigned m = e < words ? masks[e] : 0u, lo = m & 0xffffu, hi = m >> 16;
            const unsigned long long blo = __ballot(lo != 0), bhi = __ballot(hi != 0), below = (1ull << lane) - 1;
            int to = pos + __popcll(blo & below) + __popcll(bhi & below);
            if (lo) entries[to++] = (unsigned)(2 * e) << 16 | lo;
            if (hi) entries[to] = (unsigned)(2 * e + 1) << 16 | hi;
            pos += __popcll(blo) + __popcll(bhi);
        }
        __syncthreads();
        const size_t head = (size_t)n * L * 64, row = head + (size_t)u0 * 64;
        if (attend_tile(static_cast<const uint16_t *>(a.Q) + row, static_cast<const uint16_t *>(a.K) + head, static_cast<const uint16_t *>(a.V) + head,
                        a.O + row, nu, total, a.scale, a.most, room))
            return;
    }
    attend_listed(a, lists, room, L, keep, n, u0, nu);
}

// Softmax over the `keep` scores of each row: one wavefront per row.
__global__ __launch_bounds__(kRowWaves *kWave) void softmax_rows(const float *S, float *P, int keep,
                                                                  unsigned total_rows)
{
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const unsigned row = blockIdx.x * kRowWaves + wave;
    if (row >= total_rows) return;
    const float *s = S + (size_t)row * keep;
    float *p = P + (size_t)row * keep;
    constexpr int R = 8;                   // rows of up to 64 R entries stay in registers: read once, one exponential each
    if (keep <= R * kWave) {
        float v[R];
        float m = -INFINITY;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int t = lane + i * kWave;
            v[i] = t < keep ? s[t] : -INFINITY;
            m = fmaxf(m, v[i]);
        }
        m = wave_all_max(m);
        float z = 0.f;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            v[i] = __expf(v[i] - m);      // exp(-inf) = 0 beyond the row
            z += v[i];
        }
        z = wave_all_sum(z);
        const float inv = 1.f / z;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int t = lane + i * kWave;
            if (t < keep) p[t] = v[i] * inv;
        }
        return;
    }
    float m = -INFINITY;
    for (int t = lane; t < keep; t += kWave) m = fmaxf(m, s[t]);
    m = wave_all_max(m);
    float z = 0.f;
    for (int t = lane; t < keep; t += kWave) z += __expf(s[t] - m);
    z = wave_all_sum(z);
    const float inv = 1.f / z;
    for (int t = lane; t < keep; t += kWave) p[t] = __expf(s[t] - m) * inv;
}

template <typename T, int D>
hipError_t launch_rows(AttnMode mode, const dsa_shape &sh, const void *Q, const void *K, const void *V,
                       const int32_t *idx, const float *Pin, float *S, float *O, hipStream_t st)
{
    const unsigned rows = (unsigned)sh.B * sh.H * sh.L;
    const dim3 grid((rows + kRowWaves - 1) / kRowWaves), block(kRowWaves * kWave);
    // per wavefront: the padded key list and the scores / weights
    const int keep_pad = (sh.keep + kRowPad - 1) / kRowPad * kRowPad;
    const size_t lds = (size_t)kRowWaves * keep_pad * sizeof(float) * 2;
    const T *q = static_cast<const T *>(Q), *k = static_cast<const T *>(K), *v = static_cast<const T *>(V);
    if (mode == kFused) {
        auto kern = attention_rows<T, D, kFused>;
        if (hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kern), lds)) return e;
        hipLaunchKernelGGL(kern, grid, block, lds, st, q, k, v, idx, Pin, S, O, sh.L, sh.keep, keep_pad, sh.vec,
                           sh.scale, rows);
    } else if (mode == kSddmm) {
        auto kern = attention_rows<T, D, kSddmm>;
        if (hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kern), lds)) return e;
        hipLaunchKernelGGL(kern, grid, block, lds, st, q, k, v, idx, Pin, S, O, sh.L, sh.keep, keep_pad, sh.vec,
                           sh.scale, rows);
    } else {
        auto kern = attention_rows<T, D, kSpmm>;
        if (hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kern), lds)) return e;
        hipLaunchKernelGGL(kern, grid, block, lds, st, q, k, v, idx, Pin, S, O, sh.L, sh.keep, keep_pad, sh.vec,
                           sh.scale, rows);
    }
    return hipGetLastError();
}

// LDS of one workgroup of the group kernel: per wavefront 8 rows of scores and a 32-row value tile.
size_t groups_lds_bytes(const dsa_shape &sh)
{
    const size_t keep_pad = (size_t)(sh.keep + 31) / 32 * 32;
    return kGroupWaves * (9 * keep_pad * sizeof(float) + 32 * ((size_t)sh.d * 2 + 16));
}

template <int D, int MODE>
hipError_t launch_groups(const dsa_shape &sh, const void *Q, const void *K, const void *V, const int32_t *idx,
                         const float *Pin, float *S, float *O, hipStream_t st)
{
    const unsigned groups = (unsigned)sh.B * sh.H * (sh.L / 8);
    const int keep_pad = (sh.keep + 31) / 32 * 32;
    const size_t lds = groups_lds_bytes(sh);
    auto kern = attention_groups_bf16<D, MODE>;
    if (hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kern), lds)) return e;
    hipLaunchKernelGGL(kern, dim3((groups + kGroupWaves - 1) / kGroupWaves), dim3(kGroupWaves * kWave), lds, st,
                       static_cast<const uint16_t *>(Q), static_cast<const uint16_t *>(K),
                       static_cast<const uint16_t *>(V), idx, Pin, S, O, sh.L, sh.keep, keep_pad, sh.scale, groups);
    return hipGetLastError();
}

template <int D, int VEC>
hipError_t launch_units(const dsa_shape &sh, const void *Q, const void *K, const void *V, const int32_t *idx, float *O,
                        hipStream_t st)
{
    const unsigned units = (unsigned)sh.B * sh.H * (sh.L / VEC);
    const int keep_pad = (sh.keep + 31) / 32 * 32;
    const size_t lds = kGroupWaves * (unit_tile_bytes<D>() + keep_pad * sizeof(unsigned));
    auto kern = attention_units_bf16<D, VEC>;
    if (hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kern), lds)) return e;
    hipLaunchKernelGGL(kern, dim3((units + kGroupWaves - 1) / kGroupWaves), dim3(kGroupWaves * kWave), lds, st,
                       static_cast<const uint16_t *>(Q), static_cast<const uint16_t *>(K),
                       static_cast<const uint16_t *>(V), idx, O, sh.L, sh.keep, keep_pad, sh.scale, units);
    return hipGetLastError();
}

hipError_t launch_tiles(const dsa_shape &sh, int W, int most, const void *Q, const void *K, const void *V, const int32_t *idx, float *O,
                        hipStream_t st)
{
    const int tiles_per_head = (sh.L + kTileRows - 1) / kTileRows;
    const int keep_pad = (sh.keep + kRowPad - 1) / kRowPad * kRowPad;
    const size_t lds = tile_lds_bytes(sh, W, most);
    if (hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(attention_tiles_bf16), lds)) return e;
    hipLaunchKernelGGL(attention_tiles_bf16, dim3((unsigned)sh.B * sh.H * tiles_per_head), dim3(W * kWave), lds, st,
                       AttendArgs{Q, K, V, O, sh.scale, sh.d, keep_pad, most, (unsigned)lds}, idx, sh.L, sh.keep, tiles_per_head);
    return hipGetLastError();
}

template <int D>
hipError_t launch_groups_d(AttnMode mode, const dsa_shape &sh, const void *Q, const void *K, const void *V,
                           const int32_t *idx, const float *Pin, float *S, float *O, hipStream_t st)
{
    if (mode == kSddmm) return launch_groups<D, kSddmm>(sh, Q, K, V, idx, Pin, S, O, st);
    return launch_groups<D, kSpmm>(sh, Q, K, V, idx, Pin, S, O, st);
}

}  // namespace

int attention_max_keep() { return kMaxKeep; }

// The row kernel forms byte offsets inside one head (key index * bytes of a row, at most 512) in 32-bit arithmetic.
int attention_max_L() { return 1 << 22; }

hipError_t launch_attention(AttnMode mode, const dsa_shape &sh, const void *Q, const void *K,
                            const void *V, const int32_t *idx, const float *Pin, float *S, float *O,
                            hipStream_t st)
{
    if (sh.dtype == DSA_F32) {
        if (sh.d == 64) return launch_rows<float, 64>(mode, sh, Q, K, V, idx, Pin, S, O, st);
        return launch_rows<float, 128>(mode, sh, Q, K, V, idx, Pin, S, O, st);
    }
    if (sh.vec > 1 && mode == kFused) {
        if (sh.vec == 8)
            return sh.d == 64 ? launch_units<64, 8>(sh, Q, K, V, idx, O, st) : launch_units<128, 8>(sh, Q, K, V, idx, O, st);
        return sh.d == 64 ? launch_units<64, 4>(sh, Q, K, V, idx, O, st) : launch_units<128, 4>(sh, Q, K, V, idx, O, st);
    }
    if (mode == kFused && sh.vec == 1 && sh.d == 64) {
        const int W = predict_waves(sh);
        if (const int most = tile_most(sh, W)) return launch_tiles(sh, W, most, Q, K, V, idx, O, st);
    }
    if (sh.vec == 8 && groups_lds_bytes(sh) <= 144 * 1024) {
        if (sh.d == 64) return launch_groups_d<64>(mode, sh, Q, K, V, idx, Pin, S, O, st);
        return launch_groups_d<128>(mode, sh, Q, K, V, idx, Pin, S, O, st);
    }
    if (sh.d == 64) return launch_rows<uint16_t, 64>(mode, sh, Q, K, V, idx, Pin, S, O, st);
    return launch_rows<uint16_t, 128>(mode, sh, Q, K, V, idx, Pin, S, O, st);
}

hipError_t launch_attention_csr(const dsa_shape &sh, const void *Q, const void *K, const void *V,
                                const int32_t *row_ptr, const int32_t *col, float *O, hipStream_t st)
{
    const unsigned rows = (unsigned)sh.B * sh.H * sh.L;
    auto launch = [&](auto *q, auto *k, auto *v, auto d, auto waves) -> hipError_t {
        constexpr int D = decltype(d)::value, W = decltype(waves)::value;
        hipLaunchKernelGGL((attention_rows_csr<std::remove_const_t<std::remove_pointer_t<decltype(q)>>, D, W>), dim3(rows / W), dim3(W * kWave), 0, st,
                           q, k, v, row_ptr, col, O, sh.L, sh.vec, sh.scale);
        return hipGetLastError();
    };
    auto go = [&](auto *q, auto *k, auto *v) -> hipError_t {
        auto width = [&](auto d) { return sh.vec == 8 ? launch(q, k, v, d, std::integral_constant<int, 4>{}) : launch(q, k, v, d, std::integral_constant<int, 1>{}); };
        return sh.d == 64 ? width(std::integral_constant<int, 64>{}) : width(std::integral_constant<int, 128>{});
    };
    if (sh.dtype == DSA_F32) return go(static_cast<const float *>(Q), static_cast<const float *>(K), static_cast<const float *>(V));
    return go(static_cast<const uint16_t *>(Q), static_cast<const uint16_t *>(K), static_cast<const uint16_t *>(V));
}

hipError_t launch_gather_probe(const dsa_shape &sh, const void *K, const void *V, const int32_t *idx, unsigned *sink,
                               hipStream_t st)
{
    const unsigned rows = (unsigned)sh.B * sh.H * sh.L;
    const dim3 grid((rows + kRowWaves - 1) / kRowWaves), block(kRowWaves * kWave);
    const int keep_pad = (sh.keep + kRowPad - 1) / kRowPad * kRowPad;
    const size_t lds = (size_t)kRowWaves * keep_pad * sizeof(int);
    auto go = [&](auto kern, auto *k, auto *v) -> hipError_t {
        if (hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kern), lds)) return e;
        hipLaunchKernelGGL(kern, grid, block, lds, st, k, v, idx, sink, sh.L, sh.keep, keep_pad, sh.vec, rows);
        return hipGetLastError();
    };
    if (sh.dtype == DSA_F32) {
        const float *k = static_cast<const float *>(K), *v = static_cast<const float *>(V);
        return sh.d == 64 ? go(gather_probe<float, 64>, k, v) : go(gather_probe<float, 128>, k, v);
    }
    const uint16_t *k = static_cast<const uint16_t *>(K), *v = static_cast<const uint16_t *>(V);
    return sh.d == 64 ? go(gather_probe<uint16_t, 64>, k, v) : go(gather_probe<uint16_t, 128>, k, v);
}

hipError_t launch_softmax(const dsa_shape &sh, const float *S, float *P, hipStream_t st)
{
    const unsigned rows = (unsigned)sh.B * sh.H * sh.L;
    hipLaunchKernelGGL(softmax_rows, dim3((rows + kRowWaves - 1) / kRowWaves), dim3(kRowWaves * kWave),
                       0, st, S, P, sh.keep, rows);
    return hipGetLastError();
}

}  // namespace dsa
