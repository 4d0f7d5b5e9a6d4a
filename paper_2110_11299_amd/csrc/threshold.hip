// Threshold masks (paper section 3.1: the mask may be predicted "using thresholds" instead of a
// top-k search).  Unit u keeps every key whose approximate score reaches theta; a unit with none
// keeps its single best key (largest score, lower index among equals).  A unit is a query row or a
// group of vec rows whose scores are summed (section 3.3).  The count per unit varies,
// which is what the paper's equal-count constraint avoids (section 5.2), so the mask is CSR:
// row_ptr [units + 1], col [nnz], keys ascending per unit.
//
//   sweep   one wavefront per task of 16 units streams the keys once: every score is compared with theta, the outcomes are
//           the units' bitmaps, which go to the workspace together with the task's count.  The largest score per lane and
//           the word it lies in are kept beside it (half an operation per score): a unit without a key scores the 32 keys of
//           that word again and keeps the best.
//   scan    only where that many tasks make it pay (kDirectTasks): exclusive prefix sum of the counts, blocks of 1024 tasks, then the block
//           totals.
//   fill    one workgroup per task: the task's place in col (the sum of the counts before it, unless the scan has it), row_ptr,
//           and the bitmaps as keys, 64 words at a time, which leave through LDS as consecutive entries.
#include "dsa_internal.h"
#include "threshold_api.h"
#include "key_stream.h"

namespace dsa {
namespace {

constexpr int kScanBlock = 1024;        // tasks per block of the prefix sum
// Up to here every fill workgroup adds up the counts before its own (16 KB at most, from L2) instead of two more launches: a
// call with the scan and without, k = 32: 2048 tasks of L = 2048 32.0 and 28.5 us, 4096 46.7 and 45.8, 8192 80.1 and 92.7.
// Short sequences have few wavefronts to add with: L = 128 (one), 1024 tasks 14.4 and 11.3, 2048 tasks 14.8 and 16.8; L = 256
// (two), 2048 tasks 15.7 and 13.4, 4096 20.4 and 21.9; L = 512 (four), 4096 tasks 25.5 and 24.7, 8192 37.0 and 47.4.
constexpr unsigned kDirectTasks = 4096, kDirectTasksPerWave = 1024;

// Bitmap in the workspace: word w of lane l of task t at (t * NWL + w) * 64 + l (what a wavefront
// stores with one instruction is contiguous).
template <int K, int VEC>
__global__ __launch_bounds__(kWave, 4) void threshold_sweep(const int8_t *__restrict__ Qt, const int8_t *__restrict__ Kt,
                                                           unsigned *__restrict__ bitmap, int32_t *__restrict__ task_count,
                                                           int L, int theta, int tasks_per_head)
{
    const int lane = threadIdx.x;
    const int c = lane & 15, g = lane >> 4;
    const unsigned task = xcd_contiguous(blockIdx.x, gridDim.x);
    const unsigned n = task / (unsigned)tasks_per_head;
    const int u0 = (int)(task % (unsigned)tasks_per_head) * 16;
    const int Lq = stream_quarter(L), NT = Lq / 4, NWL = Lq / 32;
    const int8_t *Kh = Kt + (size_t)n * L * K;
    const int8_t *Qh = Qt + (size_t)n * L * K;
    const int G = L / VEC;                  // units of a head
    const bool unit_live = u0 + c < G;
    int tfull = NT;
#pragma unroll
    for (int q = 0; q < 4; ++q) tfull = min(tfull, max(0, min(L - q * Lq, Lq)) / 4);
    const int key_lo = g * Lq, key_lim = min(L, key_lo + Lq);

    KeyStream<K, VEC> ks;
    // no score lies beyond the limits
    const int8_t *Qu = Qh + (size_t)min(u0 + c, G - 1) * (VEC * K);
    const int limit = max(-kSweepLimit, min(theta, kSweepLimit));
    ks.start(Kh, Qu, unit_live, lane, Lq, L, -limit);
    unsigned *words = bitmap + (size_t)task * NWL * kWave + lane;
    int mine = 0, best = INT32_MIN, best_word = 0;       // best: largest score - limit so far, in word g * NWL + best_word
    for (int w = 0; w < NWL; ++w) {
        unsigned word;
        int top = INT32_MIN;
        const int nv = key_lim - (key_lo + 32 * w);      // real keys in this word
        if (8 * w + 8 + decltype(ks)::kLookahead <= tfull) {
            word = sweep_word<false>(ks, 8 * w, &top);
        } else {
            word = sweep_word<true>(ks, 8 * w, &top);
            word = nv >= 32 ? word : nv <= 0 ? 0u : word & ((1u << nv) - 1u);
        }
        words[(size_t)w * kWave] = word;
        mine += __popc(word);
        // (keys beyond L score like the last one, which shares their word if there is a real key in it)
        if (nv > 0 && top > best) { best = top; best_word = w; }
    }
    mine += __shfl_xor(mine, 16, kWave);
    mine += __shfl_xor(mine, 32, kWave);
    const bool empty = unit_live && mine == 0;
    if (__ballot(empty) != 0) {
        // the unit keeps its best key (largest score, lower index among equals): lane g takes 8 of the 32 keys
        int at = g * NWL + best_word;                    // word of the unit
#pragma unroll
        for (int off = 16; off < kWave; off <<= 1) {
            const int b2 = __shfl_xor(best, off, kWave), at2 = __shfl_xor(at, off, kWave);
            if (b2 > best || (b2 == best && at2 < at)) { best = b2; at = at2; }
        }
        int first = INT32_MAX;
#pragma unroll
        for (int i = 7; i >= 0; --i) {
            const int key = 32 * at + 8 * g + i;
            const int s = unit_key_score(reinterpret_cast<const int *>(Qu), Kh + (size_t)min(key, L - 1) * K, VEC, K / 4);
            if (key < L && s - limit == best) first = key;
        }
        first = min(first, __shfl_xor(first, 16, kWave));
        first = min(first, __shfl_xor(first, 32, kWave));
        if (empty && g == at / NWL) words[(size_t)(at % NWL) * kWave] = 1u << (first & 31);      // this lane's own word
    }
    const int all = wave_sum(g == 0 && unit_live ? max(mine, 1) : 0);
    if (lane == 0) task_count[task] = all;
}

// Exclusive prefix sums inside blocks of kScanBlock counts (in place) and the block totals.
__global__ __launch_bounds__(256) void scan_blocks(int32_t *__restrict__ count, int32_t *__restrict__ block_total, unsigned tasks)
{
    __shared__ int part[256];
    const unsigned base = blockIdx.x * kScanBlock + threadIdx.x * 4;
    int v[4], s = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[i] = base + i < tasks ? count[base + i] : 0;
        s += v[i];
    }
    part[threadIdx.x] = s;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {            // Hillis-Steele over the 256 partial sums
        const int add = threadIdx.x >= (unsigned)off ? part[threadIdx.x - off] : 0;
        __syncthreads();
        part[threadIdx.x] += add;
        __syncthreads();
    }
    int run = part[threadIdx.x] - s;                     // exclusive
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (base + i < tasks) count[base + i] = run;
        run += v[i];
    }
    if (threadIdx.x == 255) block_total[blockIdx.x] = part[255];
}

// Exclusive prefix sum of the block totals, in place: one workgroup walks them 256 at a time.
__global__ __launch_bounds__(256) void scan_totals(int32_t *__restrict__ block_total, unsigned blocks)
{
    __shared__ int part[256];
    __shared__ int carry;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (unsigned b0 = 0; b0 < blocks; b0 += 256) {
        const unsigned b = b0 + threadIdx.x;
        const int v = b < blocks ? block_total[b] : 0;
        part[threadIdx.x] = v;
        __syncthreads();
        for (int off = 1; off < 256; off <<= 1) {
            const int add = threadIdx.x >= (unsigned)off ? part[threadIdx.x - off] : 0;
            __syncthreads();
            part[threadIdx.x] += add;
            __syncthreads();
        }
        if (b < blocks) block_total[b] = carry + part[threadIdx.x] - v;
        __syncthreads();
        if (threadIdx.x == 255) carry += part[255];
        __syncthreads();
    }
}

// The words of a task in the order of its keys in col (unit by unit, word by word) are cut into NWL chunks of 64, one lane per
// word: a chunk is as much work whatever the length of a unit, so that short sequences take few wavefronts (8 of them, a unit at
// a time: L = 128, 4096 tasks, sweep to fill, 32.4 us; one: 18.0; L = 512: 35.4 and 25.1).  At most 8 share a task: N = 16,
// L = 2048: 20.3 us for the fill with 4, 17.6 with 8, 22.3 with 16, which leaves two workgroups per CU.
constexpr int kFillWaves = 8;
// Above this length one workgroup's LDS leaves no room for a second one on the CU: N = 1, L = 32768, a call with 8 wavefronts
// 555 us, with 16 437.
constexpr int kFillLong = 184, kFillWavesLong = 16;
constexpr int kFillRow = kWave + 1;     // words of LDS for one stored word of all lanes: a unit's words then lie on different banks

inline int fill_waves(int NWL) { return NWL > kFillLong ? kFillWavesLong : NWL < kFillWaves ? NWL : kFillWaves; }

// LDS: [NWL][kFillRow] the task's bitmap, then per wavefront the keys of a chunk, then a count per chunk and a sum per wavefront.
__host__ __device__ inline size_t fill_bitmap_bytes(int NWL) { return ((size_t)NWL * kFillRow * 4 + 15) / 16 * 16; }
inline size_t fill_lds_bytes(int NWL)
{
    return fill_bitmap_bytes(NWL) + fill_waves(NWL) * 32 * kWave * sizeof(uint16_t) + (NWL + fill_waves(NWL)) * sizeof(int);
}

__global__ __launch_bounds__(kFillWavesLong *kWave) void threshold_fill(const unsigned *__restrict__ bitmap,
                                                      const int32_t *__restrict__ task_count,
                                                      const int32_t *__restrict__ block_total,
                                                      int32_t *__restrict__ row_ptr, int32_t *__restrict__ col,
                                                      long long col_capacity, int L, int vec, int tasks_per_head,
                                                      unsigned units)
{
    extern __shared__ __align__(16) unsigned words[];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int T = blockDim.x, waves = T / kWave;
    const unsigned task = xcd_contiguous(blockIdx.x, gridDim.x);
    const int G = L / vec;
    const unsigned n = task / (unsigned)tasks_per_head;
    const int u0 = (int)(task % (unsigned)tasks_per_head) * 16, nu = min(16, G - u0);
    const int Lq = stream_quarter(L), NWL = Lq / 32, NW = 4 * NWL;
    uint16_t *keys = reinterpret_cast<uint16_t *>(reinterpret_cast<char *>(words) + fill_bitmap_bytes(NWL));
    int *s_count = reinterpret_cast<int *>(keys + waves * 32 * kWave);
    int *s_part = s_count + NWL;
    keys += wave * 32 * kWave;
    const unsigned *stored = bitmap + (size_t)task * NWL * kWave;
    for (int e = tid; e < NWL * kWave; e += T) words[(e / kWave) * kFillRow + lane] = stored[e];
    // entries before the task's
    int before = 0;
    if (block_total) {
        before = task_count[task] + block_total[task / kScanBlock];
    } else {
        for (unsigned t = tid; t < task; t += T) before += task_count[t];
        before = wave_sum(before);
        if (lane == 0) s_part[wave] = before;
    }
    __syncthreads();
    if (!block_total) {
        before = 0;
        for (int w = 0; w < waves; ++w) before += s_part[w];
    }
    // word e of the task: word W of unit c, which is quarter W / NWL, word W % NWL of lane 16 * quarter + c
    // (quotients below 16 of numbers below 2^14: a product with the reciprocal is off by less than 2^-19, and (x + 1/2) / y is
    // at least 2^-11 away from the next whole number)
    const float per_unit = 1.f / (float)NW, per_quarter = 1.f / (float)NWL;
    auto unit_of = [&](int e) { return (int)(((float)e + 0.5f) * per_unit); };
    auto word_of = [&](int c, int W) -> unsigned {
        const int q = (int)(((float)W + 0.5f) * per_quarter), w = W - q * NWL;
        return c < nu ? words[w * kFillRow + 16 * q + c] : 0u;
    };
    for (int j = wave; j < NWL; j += waves) {
        const int e = j * kWave + lane, c = unit_of(e);
        const int count = wave_sum(__popc(word_of(c, e - c * NW)));
        if (lane == 0) s_count[j] = count;
    }
    __syncthreads();
    for (int j = wave; j < NWL; j += waves) {
        int sum = 0;
        for (int i = lane; i < j; i += kWave) sum += s_count[i];
        const long long start = before + wave_sum(sum);
        const int e = j * kWave + lane, c = unit_of(e), W = e - c * NW;
        unsigned m = word_of(c, W);
        int total;
        const int end = wave_incl_scan(__popc(m), lane, &total);
        int rank = end - __popc(m);
        const unsigned u = n * (unsigned)G + u0 + c;
        if (c < nu && W == 0) row_ptr[u] = (int32_t)(start + rank);
        if (c == nu - 1 && W == NW - 1 && u + 1 == units) row_ptr[units] = (int32_t)(start + end);       // nnz
        const int key1 = 32 * W - 1;
        while (m) {
            keys[rank++] = (uint16_t)(key1 + __ffs(m));
            m &= m - 1u;
        }
        wave_lds_sync();
        int32_t *out = col + start;
        const long long room = col_capacity - start;      // entries beyond the capacity are left out
        for (int t = lane; t < total; t += kWave)
            if (t < room) out[t] = keys[t];
        wave_lds_sync();
    }
}

template <int K, int VEC>
hipError_t launch_threshold_kv(const dsa_shape &sh, const int8_t *Qt, const int8_t *Kt, int theta, int32_t *row_ptr,
                              int32_t *col, long long col_capacity, void *ws, hipStream_t st)
{
    const int tasks_per_head = (sh.L / VEC + 15) / 16;
    const unsigned tasks = (unsigned)sh.B * sh.H * tasks_per_head;
    const unsigned units = (unsigned)sh.B * sh.H * (sh.L / VEC);
    const size_t bitmap_words = (size_t)tasks * (stream_quarter(sh.L) / 32) * kWave;
    unsigned *bitmap = static_cast<unsigned *>(ws);
    int32_t *task_count = reinterpret_cast<int32_t *>(bitmap + bitmap_words);
    const int NWL = stream_quarter(sh.L) / 32;
    const unsigned direct = min(kDirectTasks, kDirectTasksPerWave * fill_waves(NWL));
    int32_t *block_total = tasks > direct ? task_count + tasks : nullptr;
    hipLaunchKernelGGL((threshold_sweep<K, VEC>), dim3(tasks), dim3(kWave), 0, st, Qt, Kt, bitmap, task_count, sh.L, theta,
                       tasks_per_head);
    if (block_total) {
        const unsigned blocks = (tasks + kScanBlock - 1) / kScanBlock;
        hipLaunchKernelGGL(scan_blocks, dim3(blocks), dim3(256), 0, st, task_count, block_total, tasks);
        hipLaunchKernelGGL(scan_totals, dim3(1), dim3(256), 0, st, block_total, blocks);
    }
    const size_t lds = fill_lds_bytes(NWL);
    if (hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(threshold_fill), lds)) return e;
    hipLaunchKernelGGL(threshold_fill, dim3(tasks), dim3(fill_waves(NWL) * kWave), lds, st, bitmap, task_count, block_total, row_ptr,
                       col, col_capacity, sh.L, VEC, tasks_per_head, units);
    return hipGetLastError();
}

template <int K>
hipError_t launch_threshold_k(const dsa_shape &sh, const int8_t *Qt, const int8_t *Kt, int theta, int32_t *row_ptr,
                              int32_t *col, long long col_capacity, void *ws, hipStream_t st)
{
    if (sh.vec == 1) return launch_threshold_kv<K, 1>(sh, Qt, Kt, theta, row_ptr, col, col_capacity, ws, st);
    if (sh.vec == 4) return launch_threshold_kv<K, 4>(sh, Qt, Kt, theta, row_ptr, col, col_capacity, ws, st);
    return launch_threshold_kv<K, 8>(sh, Qt, Kt, theta, row_ptr, col, col_capacity, ws, st);
}

}  // namespace

bool threshold_supported(const dsa_shape &sh)
{
    return (sh.vec == 1 || sh.vec == 4 || sh.vec == 8) && (sh.k == 16 || sh.k == 32 || sh.k == 64);
}

size_t threshold_workspace_bytes(const dsa_shape &sh)
{
    const size_t tasks = (size_t)sh.B * sh.H * ((sh.L / sh.vec + 15) / 16);
    const size_t units = (size_t)sh.B * sh.H * (sh.L / sh.vec);
    const size_t blocks = (units + kScanBlock - 1) / kScanBlock;
    // (the counts are one per task; callers have been told to bring room for one per unit, and the figure stays)
    return sizeof(unsigned) * tasks * (stream_quarter(sh.L) / 32) * kWave + sizeof(int32_t) * (units + blocks);
}

hipError_t launch_predict_threshold(const dsa_shape &sh, const int8_t *Qt, const int8_t *Kt, int theta,
                                    int32_t *row_ptr, int32_t *col, long long col_capacity, void *ws, hipStream_t st)
{
    if (sh.k == 16) return launch_threshold_k<16>(sh, Qt, Kt, theta, row_ptr, col, col_capacity, ws, st);
    if (sh.k == 32) return launch_threshold_k<32>(sh, Qt, Kt, theta, row_ptr, col, col_capacity, ws, st);
    return launch_threshold_k<64>(sh, Qt, Kt, theta, row_ptr, col, col_capacity, ws, st);
}

}  // namespace dsa
