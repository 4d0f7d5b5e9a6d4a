// Launcher of the mask predictor (predict_split.h) and the approximate-score contraction of paper
// section 3.1 by itself: row maxima of S~ = Q~ K~^T, and the int8 matrix-core yardstick.
#include "dsa_internal.h"
#include "predict_api.h"
#include "split_plan.h"
#include "wave_select.h"

namespace dsa {
namespace {

// Row maximum of the approximate scores with the int8 matrix cores: the contraction with the
// smallest consumer that still looks at every score.  A wavefront keeps 64 query rows as two B
// operands of v_mfma_i32_32x32x32_i8 and sweeps its share of the keys 32 at a time as the A
// operand, so each lane ends up with one query column per operand and 16 key rows per tile: the
// running maximum is a per-lane scalar.  Key tiles are prefetched several tiles ahead into a
// register ring, and the maxima of tile t are taken (two scores per v_max3) while the matrix
// core works on tile t+1.  KSPLIT wavefronts share one 64-row query tile and split the keys, so
// that a SIMD holds several wavefronts and one's v_max3 stream fills the other's matrix-core
// time; they combine through LDS at the end.  A workgroup is always 8 wavefronts: 8 / KSPLIT
// query tiles times KSPLIT key shares.
// (With 512 threads, at most 256 registers per lane, the compiler gives the matrix core plain
// VGPR destinations that v_max3 can read directly.)
template <int KSTEPS, int KSPLIT, int NQ>   // k padded to 32 * KSTEPS; NQ blocks of 32 query rows per wavefront
__global__ __launch_bounds__(512) void rowmax_mfma(
    const int8_t *__restrict__ Qt, const int8_t *__restrict__ Kt, int32_t *__restrict__ rowmax, int L, int k,
    unsigned N)
{
    constexpr int PD = 8 / KSTEPS;                       // prefetch depth in tiles (KSTEPS <= 4)
    constexpr int QR = 32 * NQ;                          // query rows per wavefront
    constexpr int QSLOTS = 8 / KSPLIT;                   // query tiles per workgroup of 8 wavefronts
    __shared__ int part[8][QR];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int col = lane & 31, half = lane >> 5;
    const int qslot = wave / KSPLIT, ks = wave % KSPLIT;
    const unsigned qtiles_per_head = (L + QR - 1) / QR;
    const unsigned qtile = xcd_contiguous(blockIdx.x, gridDim.x) * QSLOTS + qslot;
    const bool live = qtile < N * qtiles_per_head;
    const unsigned n = live ? qtile / qtiles_per_head : 0;
    const int i0 = live ? (int)(qtile % qtiles_per_head) * QR : 0;
    const int8_t *Qh = Qt + (size_t)n * L * k, *Kh = Kt + (size_t)n * L * k;

    // operand piece of this lane: 16 consecutive c at 32*step + 16*half.  Beyond k (and, for
    // queries, beyond L) the query piece is zero, so the key piece there may hold anything and is
    // read from offset 0.  Key rows beyond L are read from row L-1 and masked at the end.
    int coff[KSTEPS];
    v4i qop[NQ][KSTEPS];
#pragma unroll
    for (int s = 0; s < KSTEPS; ++s) {
        const int c = 32 * s + 16 * half;
        coff[s] = c < k ? c : 0;
#pragma unroll
        for (int h = 0; h < NQ; ++h) {
            const int qi = i0 + 32 * h + col;
            qop[h][s] = (qi < L && c < k) ? *reinterpret_cast<const v4i *>(Qh + (size_t)qi * k + c) : v4i{0, 0, 0, 0};
        }
    }
    const int T = (L + 31) / 32;                       // key tiles in all
    const int Tper = (T + KSPLIT - 1) / KSPLIT;
    const int ta = ks * Tper, tb = min(T, ta + Tper);  // this wavefront's tiles
    auto load_tile = [&](int t, v4i (&dst)[KSTEPS]) {
        const int8_t *row = Kh + (size_t)min(32 * t + col, L - 1) * k;
#pragma unroll
        for (int s = 0; s < KSTEPS; ++s) dst[s] = *reinterpret_cast<const v4i *>(row + coff[s]);
    };
    v4i ring[PD][KSTEPS];
#pragma unroll
    for (int p = 0; p < PD; ++p) load_tile(min(ta + p, T - 1), ring[p]);

    int m[NQ];
    v16i prev[NQ];         // scores of the previous tile, reduced while the next one is computed
#pragma unroll
    for (int h = 0; h < NQ; ++h) {
        m[h] = INT32_MIN;
#pragma unroll
        for (int r = 0; r < 16; ++r) prev[h][r] = INT32_MIN;
    }
    auto step = [&](v4i (&kop)[KSTEPS]) {
        v16i cur[NQ];
#pragma unroll
        for (int h = 0; h < NQ; ++h) {
            cur[h] = v16i{0};
#pragma unroll
            for (int s = 0; s < KSTEPS; ++s)
                cur[h] = __builtin_amdgcn_mfma_i32_32x32x32_i8(kop[s], qop[h][s], cur[h], 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
#pragma unroll
            for (int h = 0; h < NQ; ++h) m[h] = max(max(prev[h][r], prev[h][r + 1]), m[h]);
        }
#pragma unroll
        for (int h = 0; h < NQ; ++h) prev[h] = cur[h];
    };
    // all tiles but the last of the sweep hold only real keys; the ring slot of tile t is (t - ta) % PD
    int t = ta;
    for (; t + PD <= tb - 1; t += PD) {
#pragma unroll
        for (int p = 0; p < PD; ++p) {
            step(ring[p]);
            load_tile(min(t + p + PD, T - 1), ring[p]);
            // keep the refill of slot p here, PD tiles ahead of its use: left alone, the scheduler
            // gathers all refills at the end of the unrolled body, right before they are needed
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int p = 0; p < PD; ++p)
        if (t + p < tb) step(ring[p]);      // the rest; prev ends up as tile tb-1
    // that tile may reach past L: register r of this lane is key row 8*(r/4) + 4*half + r%4 of it
    if (ta < tb) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            if (32 * (tb - 1) + 8 * (r / 4) + 4 * half + (r % 4) < L) {
#pragma unroll
                for (int h = 0; h < NQ; ++h) m[h] = max(m[h], prev[h][r]);
            }
        }
    }
#pragma unroll
    for (int h = 0; h < NQ; ++h) {
        m[h] = max(m[h], __shfl_xor(m[h], 32, kWave));
        if (half == 0) part[wave][32 * h + col] = m[h];
    }
    __syncthreads();
    if (ks == 0 && live) {
        for (int r = lane; r < QR; r += kWave) {
            int best = part[wave][r];
#pragma unroll
            for (int j = 1; j < KSPLIT; ++j) best = max(best, part[wave + j][r]);
            if (i0 + r < L) rowmax[(size_t)n * L + i0 + r] = best;
        }
    }
}

}  // namespace

int predict_max_L() { return 32768; }

int predict_waves(const dsa_shape &sh)
{
    const SplitPlan p = split_plan(sh, split_pairs_exist(sh.k, sh.vec > 1));
    return p.UT == 1 ? p.W : 0;
}

size_t predict_workspace_bytes(const dsa_shape &) { return 0; }

hipError_t launch_predict(const dsa_shape &sh, const int8_t *Qt, const int8_t *Kt, int32_t *idx, void *,
                          const AttendPtrs *attend, bool *attended, hipStream_t st)
{
    switch (sh.k) {
    case 16: return launch_split_k16(sh, Qt, Kt, idx, attend, attended, st);
    case 32: return launch_split_k32(sh, Qt, Kt, idx, attend, attended, st);
    case 48: return launch_split_k48(sh, Qt, Kt, idx, attend, attended, st);
    case 64: return launch_split_k64(sh, Qt, Kt, idx, attend, attended, st);
    case 128: return launch_split_k128(sh, Qt, Kt, idx, attend, attended, st);
    default: return launch_split_any(sh, Qt, Kt, idx, attend, attended, st);
    }
}

// Nothing but v_mfma_i32_32x32x32_i8: four independent accumulation chains per wavefront, no memory
// traffic inside the loop.  Measures the int8 matrix-core rate the chip sustains at its own clocks,
// the yardstick for rowmax_mfma next to the published peak.
__global__ __launch_bounds__(256) void mfma_i8_stream(int iters, int32_t *__restrict__ sink)
{
    v4i a, b;
#pragma unroll
    for (int i = 0; i < 4; ++i) { a[i] = 0x01020304 * (i + 1) + (int)threadIdx.x; b[i] = 0x04030201 * (i + 1) - (int)threadIdx.x; }
    v16i c0 = {0}, c1 = {0}, c2 = {0}, c3 = {0};
    for (int i = 0; i < iters; ++i) {
        c0 = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c0, 0, 0, 0);
        c1 = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c1, 0, 0, 0);
        c2 = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c2, 0, 0, 0);
        c3 = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c3, 0, 0, 0);
    }
    sink[blockIdx.x * 256 + threadIdx.x] = c0[0] + c1[1] + c2[2] + c3[3];
}

template <int KSTEPS, int NQ>
hipError_t launch_rowmax_q(const dsa_shape &sh, const int8_t *Qt, const int8_t *Kt, int32_t *rowmax, hipStream_t st)
{
    const unsigned N = (unsigned)sh.B * sh.H;
    const unsigned qtiles = N * ((sh.L + 32 * NQ - 1) / (32 * NQ));
    // enough wavefronts for a few per SIMD (1024 SIMDs), but at least 8 key tiles each
    const int tiles = (sh.L + 31) / 32;
    int ksplit = 1;
    while (ksplit < 8 && (size_t)qtiles * ksplit < 2048 && tiles / (2 * ksplit) >= 8) ksplit *= 2;
    const unsigned slots = 8 / ksplit;
    const dim3 grid((qtiles + slots - 1) / slots), block(512);
    switch (ksplit) {
    case 1: hipLaunchKernelGGL((rowmax_mfma<KSTEPS, 1, NQ>), grid, block, 0, st, Qt, Kt, rowmax, sh.L, sh.k, N); break;
    case 2: hipLaunchKernelGGL((rowmax_mfma<KSTEPS, 2, NQ>), grid, block, 0, st, Qt, Kt, rowmax, sh.L, sh.k, N); break;
    case 4: hipLaunchKernelGGL((rowmax_mfma<KSTEPS, 4, NQ>), grid, block, 0, st, Qt, Kt, rowmax, sh.L, sh.k, N); break;
    default: hipLaunchKernelGGL((rowmax_mfma<KSTEPS, 8, NQ>), grid, block, 0, st, Qt, Kt, rowmax, sh.L, sh.k, N); break;
    }
    return hipGetLastError();
}

template <int KSTEPS>
hipError_t launch_rowmax_k(const dsa_shape &sh, const int8_t *Qt, const int8_t *Kt, int32_t *rowmax, hipStream_t st)
{
    // 128 query rows per wavefront (one key operand feeds four MFMAs) when that still leaves enough
    // wavefronts to fill the chip and k is short enough for the registers; else 64
    const size_t rows = (size_t)sh.B * sh.H * sh.L;
    if (KSTEPS <= 2 && rows >= 65536) return launch_rowmax_q<KSTEPS, 4>(sh, Qt, Kt, rowmax, st);
    return launch_rowmax_q<KSTEPS, 2>(sh, Qt, Kt, rowmax, st);
}

hipError_t launch_rowmax(const dsa_shape &sh, const int8_t *Qt, const int8_t *Kt, int32_t *rowmax,
                         hipStream_t st)
{
    switch ((sh.k + 31) / 32) {
    case 1: return launch_rowmax_k<1>(sh, Qt, Kt, rowmax, st);
    case 2: return launch_rowmax_k<2>(sh, Qt, Kt, rowmax, st);
    case 3: return launch_rowmax_k<3>(sh, Qt, Kt, rowmax, st);
    default: return launch_rowmax_k<4>(sh, Qt, Kt, rowmax, st);
    }
}

hipError_t launch_mfma_i8_stream(int blocks, int iters, int32_t *sink, hipStream_t st)
{
    hipLaunchKernelGGL(mfma_i8_stream, dim3(blocks), dim3(256), 0, st, iters, sink);
    return hipGetLastError();
}

}  // namespace dsa
