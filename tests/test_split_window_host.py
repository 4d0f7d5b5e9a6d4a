"""Where the predictor's histogram has its bins (csrc/split_plan.h), asked on the CPU: a window of some width for every plan, which has the
thresholds of normally distributed scores inside."""
import subprocess
from pathlib import Path

import numpy as np

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
