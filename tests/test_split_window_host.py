"""Where the predictor's histogram has its bins (csrc/split_plan.h), asked on the CPU: a window of some width for every plan, which has the
thresholds of normally distributed scores inside; and what the thresholds that come of it cost, with the kernel's own arithmetic (csrc/split_bounds.h), for
keys whose norms vary or that lie in clusters."""
import subprocess
from pathlib import Path

import numpy as np
import pytest

ROOT = Path(__file__).resolve().parent.parent
CSRC = ROOT / "paper_2110_11299_amd" / "csrc"

# a line "N L k keep vec" in; words and buckets per lane, targets, the window out
PROGRAM = r"""
#include "split_plan.h"
#include <cstdio>
int main()
{
    dsa_shape s{};
    s.B = 1; s.d = 64; s.dtype = DSA_BF16; s.scale = 1.f;
    while (scanf("%d %d %d %d %d", &s.H, &s.L, &s.k, &s.keep, &s.vec) == 5) {
        const dsa::SplitPlan p = dsa::split_plan(s, dsa::split_pairs_exist(s.k, s.vec > 1));
        printf("%d %d %d %d %.9g %.9g\n", p.NW, p.NB, p.target_l, p.target_h, p.low, p.high);
    }
}
"""


def test_thresholds_lie_in_the_window(tmp_path):
    (tmp_path / "window.hip").write_text(PROGRAM)
    subprocess.run(["/opt/rocm/bin/hipcc", "--offload-host-only", "-O2", "-std=c++17", "-w", f"-I{CSRC}", f"-I{ROOT / 'include'}", str(tmp_path / "window.hip"),
                    "-o", str(tmp_path / "window")], check=True)
    shapes = [(n, L, k, keep, vec) for n in (1, 64) for L in (1, 7, 64, 128, 129, 256, 500, 513, 1000, 2048, 4096, 5000, 8192, 16384, 32768) for k in (16, 64)
              for vec in (1, 8) if L % vec == 0 for keep in sorted({1, max(1, L // 100), max(1, L // 20), max(1, L // 8), max(1, L // 2), max(1, L - 1), L})]
    out = subprocess.run([str(tmp_path / "window")], input="".join("%d %d %d %d %d\n" % s for s in shapes), capture_output=True, text=True, check=True).stdout
    rng = np.random.Generator(np.random.Philox(7))
    for shape, line in zip(shapes, out.splitlines(), strict=True):
        n, L, k, keep, vec = shape
        NW, NB, target_l, target_h = map(int, line.split()[:4])
        low, high = map(float, line.split()[4:])
        assert -1.0 <= low < high <= 2.0, shape
        if L < 500 or n > 1:
            continue
        # buckets of a range, as many keys in each as the kernel puts there
        scores = rng.standard_normal((32, L))
        if NW > 1:
            Lr = 32 * NW
            w = np.arange(Lr) // 32
            bucket = np.arange(Lr) % 16 + (16 * (w % 2) if NB == 32 else 0)
            full = scores[:, :L // Lr * Lr].reshape(32, -1, Lr)
            scores = np.stack([full[:, :, bucket == b].max(axis=2) for b in range(NB)], axis=2).reshape(32, -1)
        share = scores.shape[1] / (L if NW == 1 else NB * L / (32 * NW))
        mean, least = scores.mean(axis=1), scores.min(axis=1)
        ordered = -np.sort(-scores, axis=1)
        for target in (target_l, target_h):
            at = int(round(target * share)) - 1
            if 0 <= at < scores.shape[1]:
                place = (ordered[:, at] - mean) / (mean - least)
                inside = (place >= low - 1e-6) & (place <= high + 1e-6)
                assert inside.mean() >= 0.9, (shape, target, low, high, place.min(), place.max())


# The bounds and the sweeps of a unit, as predict_split has them.  A first line "mode N L k keep vec units" and the scores in binary; mode 0 has the bins over
# all maxima, from the smallest to three times the distance to the mean, and no second histogram.  Out: sweeps and histograms of a workgroup, the most of any of its units,
# and the keys of the longest band, on average.
REPLAY = r"""
#include "split_plan.h"
#include "split_bounds.h"
#include <algorithm>
#include <climits>
#include <cstdio>
#include <vector>
using namespace dsa;
int main()
{
    int mode, units;
    dsa_shape s{};
    s.B = 1; s.d = 64; s.dtype = DSA_F32; s.scale = 1.f;
    if (scanf("%d %d %d %d %d %d %d", &mode, &s.H, &s.L, &s.k, &s.keep, &s.vec, &units) != 7 || getchar() != '\n') return 1;
    const SplitPlan p = split_plan(s, split_pairs_exist(s.k, s.vec > 1));
    const int L = s.L, Lr = 32 * p.NW, ranges = 4 * p.W, U = 16 * p.UT;
    const int cap = 16 * (s.vec == 1 && p.UT == 1 && p.NW > 1 ? 32 : 24), smax = s.vec * s.k * 16384, smin = -s.vec * s.k * 16256;
    const bool again = mode && split_bins_again(s.k, s.vec > 1, p.NW);
    double sweeps = 0, histograms = 0, bands = 0;
    int most_sweeps = 0, most_histograms = 0, longest = 0;
    std::vector<int> x(L);
    for (int u = 0; u < units; ++u) {
        if (fread(x.data(), 4, L, stdin) != (size_t)L) return 2;
        std::vector<int> maxima, full;          // all of them, and those of ranges that do not end beyond the head
        for (int h = 0; h * Lr < L; ++h) {
            std::vector<int> b(p.NB, INT_MIN);
            for (int r = 0; r < Lr && h * Lr + r < L; ++r) {
                const int w = r / 32, j = r % 32 / 4, at = p.NW == 1 ? r : (p.NB == 32 ? 16 * (w % 2) : 0) + 4 * (2 * (j / 4) + j % 2) + r % 4;
                b[at] = std::max(b[at], x[h * Lr + r]);
            }
            for (int v : b)
                if (v != INT_MIN) {
                    maxima.push_back(v);
                    if (p.NW == 1 || h * Lr + Lr <= L) full.push_back(v);
                }
        }
        const int least = *std::min_element(full.begin(), full.end()), added = p.NW == 1 ? L : p.NB * (L / Lr);
        double sum = 0;
        for (int v : full) sum += v;
        SplitBins bins = window_bins((float)(sum / added), least, mode ? p.low : -1.f, mode ? p.high : 2.f, mode && !again);
        if (!mode) bins.base = least;
        int tl = 0, th = 0, round = 1;
        for (;; ++round) {
            int in[kBins] = {}, edge_h = kBins, edge_l = -1, count_h = 0, count_l = 0, suffix = 0;
            for (int v : maxima)
                if (split_bin(bins, v) >= 0) ++in[split_bin(bins, v)];
            for (int e = kBins - 1; e >= 0; --e) {
                suffix += in[e];
                if (suffix <= p.target_h) { edge_h = e; count_h = suffix; }
                if (suffix >= p.target_l && edge_l < 0) { edge_l = e; count_l = suffix; }
            }
            const bool below = edge_l < 0, above = edge_h == kBins;
            if (round > 1 && above) return 3;
            tl = bins.base + (std::max(edge_l, 0) << bins.shift);
            th = bins.base + (edge_h << bins.shift);
            if (round == 1) {
                if (below) tl = least;
                if (above) th = smax + 1;
                if (!again || !(below || above) || !split_crowded((below ? added : count_l) - count_h, p.target_l, p.target_h)) break;
            } else if (round == kBinRounds || bins.shift == 0 || th - tl > kBins / 4 << bins.shift || !split_crowded(count_l - count_h, p.target_l, p.target_h)) break;
            bins = bracket_bins(round == 1 && below ? *std::min_element(maxima.begin(), maxima.end()) : tl,
                                round == 1 && above ? *std::max_element(maxima.begin(), maxima.end()) + 1 : th);
        }
        SplitBracket b{tl, std::min(std::max(th, tl + 1), smax + 1), smin, smax + 1, L, 0};
        int tries = 0, nl, nh;
        for (;; ++tries) {
            if (tries > 100) return 4;
            nl = nh = 0;
            for (int v : x) { nl += v >= b.tl; nh += v >= b.th; }
            if (b.good(nl, nh, s.keep, cap)) break;
            b.move(nl, nh, s.keep, cap, tries);
        }
        most_sweeps = std::max(most_sweeps, tries + 1);
        most_histograms = std::max(most_histograms, round);
        longest = std::max(longest, nh == s.keep || b.th - b.tl == 1 ? 0 : nl - nh);
        if (u % U == U - 1) {
            sweeps += most_sweeps; histograms += most_histograms; bands += longest;
            most_sweeps = most_histograms = longest = 0;
        }
    }
    printf("%f %f %f\n", sweeps / (units / U), histograms / (units / U), bands / (units / U));
}
"""


@pytest.fixture(scope="module")
def replay(tmp_path_factory):
    at = tmp_path_factory.mktemp("replay")
    (at / "replay.hip").write_text(REPLAY)
    subprocess.run(["/opt/rocm/bin/hipcc", "--offload-host-only", "-O2", "-std=c++17", "-w", f"-I{CSRC}", f"-I{ROOT / 'include'}", str(at / "replay.hip"),
                    "-o", str(at / "replay")], check=True)

    def run(mode, N, L, k, keep, vec, scores):
        head = "%d %d %d %d %d %d %d\n" % (mode, N, L, k, keep, vec, len(scores))
        out = subprocess.run([str(at / "replay")], input=head.encode() + scores.tobytes(), capture_output=True, check=True, timeout=60).stdout
        return tuple(map(float, out.split()))
    return run


def codes_of(rng, L, k, kind, queries):
    """Low-rank codes of a head's queries and keys, whose norms vary, or that lie in clusters."""
    rank = 8 if L <= 256 else 32

    def signal(n):
        return rng.standard_normal((n, rank)) @ (rng.standard_normal((rank, 64)) * rank ** -0.5) + 0.1 * rng.standard_normal((n, 64))
    R = rng.standard_normal((64, k)) * k ** -0.5
    Q, K = signal(queries), signal(L)
    high = {"one": 1, "1 %": max(1, L // 100), "5 %": L // 20}.get(kind, 0)
    K[rng.choice(L, high, replace=False)] *= 4.0                    # keys of four times the norm
    if kind == "log-normal":
        K *= np.exp(0.8 * rng.standard_normal((L, 1)))
    if kind == "clusters":
        K = 2.0 * signal(8)[rng.integers(0, 8, L)] + 0.3 * K
    if kind == "sinks":                                             # a few keys that every query has high scores with
        at, way = rng.choice(L, max(1, L // 33), replace=False), 2.0 * signal(1)
        K[at] = way + 0.3 * K[at]
        Q = 0.5 * Q + way
    return [np.clip(np.rint(x @ R * (127.0 / np.abs(x @ R).max())), -127, 127) for x in (Q, K)]


# ranges of one word (1, 4 and 8 wavefronts), of 2 to 16, that end at the head and beyond, with one tile and two, groups at k = 16
@pytest.mark.parametrize("N,L,k,keep,vec", [(2, 128, 16, 13, 1), (2, 256, 16, 26, 1), (96, 384, 32, 38, 1), (96, 512, 32, 26, 1), (96, 512, 32, 51, 1), (200, 500, 32, 25, 4),
                                            (96, 512, 64, 256, 8), (16, 777, 32, 39, 1), (48, 1000, 32, 50, 4), (64, 2000, 16, 200, 4), (2, 2104, 32, 32, 1), (2, 896, 32, 36, 1), (2, 1032, 64, 20, 1), (2, 3680, 16, 40, 1), (64, 2048, 32, 102, 8),
                                            (16, 4096, 32, 41, 1), (16, 4096, 32, 205, 1), (16, 4096, 32, 205, 8), (16, 4096, 32, 410, 1), (16, 4096, 64, 82, 1), (2, 7792, 32, 145, 8),
                                            (4, 8192, 32, 410, 1), (16, 8192, 64, 82, 8), (4, 16384, 64, 164, 1)])
def test_sweeps(replay, N, L, k, keep, vec):
    """Workgroups sweep their keys no more often than with bins over all maxima, and bands get no longer but within what is scored at once."""
    rng = np.random.Generator(np.random.Philox(L + keep))
    for kind in ("plain", "one", "1 %", "5 %", "log-normal", "clusters", "sinks"):
        Qt, Kt = codes_of(rng, L, k, kind, 96 * vec)
        scores = (Qt.reshape(96, vec, k).sum(axis=1) @ Kt.T).astype(np.int32)
        sweeps, histograms, band = replay(1, N, L, k, keep, vec, scores)
        sweeps_all, _, band_all = replay(0, N, L, k, keep, vec, scores)
        assert sweeps <= sweeps_all, kind
        assert band <= max(1.1 * band_all, 96.0), kind                              # (six slots of 16)
        assert histograms <= 2.5, kind
        if kind == "plain":
            assert sweeps == histograms == 1.0 and band < band_all
