"""Which calls of the fine-grained bf16 attention go over the union of 16 rows' lists: the rule itself (csrc/tile_attend.h with the plan of
csrc/split_plan.h), built for the host and asked on the CPU."""
import subprocess
from pathlib import Path

import pytest

from test_gpu_tiles import LINES

ROOT = Path(__file__).resolve().parent.parent
CSRC = ROOT / "paper_2110_11299_amd" / "csrc"

# a line "B H L d k keep vec dtype scale" in; wavefronts per tile of the plan, longest union (0: row by row), bytes of LDS out
PROGRAM = r"""
#include "split_plan.h"
#include "tile_attend.h"
#include <cstdio>
int main()
{
    dsa_shape s{};
    while (scanf("%d %d %d %d %d %d %d %d %f", &s.B, &s.H, &s.L, &s.d, &s.k, &s.keep, &s.vec, &s.dtype, &s.scale) == 9) {
        const dsa::SplitPlan p = dsa::split_plan(s, dsa::split_pairs_exist(s.k, s.vec > 1));
        const int W = p.UT == 1 ? p.W : 0, most = dsa::tile_most(s, W);
        printf("%d %d %zu\n", W, most, most ? dsa::tile_lds_bytes(s, W, most) : (size_t)0);
    }
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    at = tmp_path_factory.mktemp("rule")
    (at / "rule.hip").write_text(PROGRAM)
    subprocess.run(["/opt/rocm/bin/hipcc", "--offload-host-only", "-O2", "-std=c++17", "-w", f"-I{CSRC}", f"-I{ROOT / 'include'}", str(at / "rule.hip"),
                    "-o", str(at / "rule")], check=True)

    def run(shapes):
        """shapes: (N, L, k, keep), or with the scale, or scale, type and d behind it -> (wavefronts or, of two tiles, 0, longest union, LDS bytes) of each"""
        full = [(*s, *(0.125, 1, 64)[len(s) - 4:]) for s in shapes]
        lines = "".join(f"1 {n} {L} {d} {k} {keep} 1 {dtype} {scale}\n" for n, L, k, keep, scale, dtype, d in full)
        out = subprocess.run([str(at / "rule")], input=lines, capture_output=True, text=True, check=True).stdout.split()
        return [tuple(map(int, out[i:i + 3])) for i in range(0, len(out), 3)]
    return run


def test_no_scale(ask):
    """With a scale of 0 the exponent of a key that is not kept would be 0 * -infinity."""
    for shape in ((16, 4096, 32, 410), (256, 256, 16, 26), (2, 16384, 32, 1366)):
        with_scale, negative, without, minus = ask([shape, (*shape, -0.125), (*shape, 0.0), (*shape, -0.0)])
        assert with_scale[1] > 0 and negative[1] == with_scale[1]
        assert without[1] == 0 and minus[1] == 0


def test_lines(ask):
    for shape in LINES:
        n, L, k, keep = shape
        on, off = ask([shape, (n, L, k, keep - 1)])
        assert on[1] >= min(L, 16 * keep) and off[1] == 0, shape
        assert on[2] <= 128 * 1024


# from two and three rounds of wavefronts on, (N, L, k, keep): the line, with one key less row by row; and with fewer wavefronts
@pytest.mark.parametrize("shape,fewer", [((70, 700, 32, 70), 69), ((64, 1024, 16, 79), 63), ((16, 2048, 64, 137), 15), ((11, 3000, 32, 188), 10), ((8, 4096, 32, 256), 7),
                                         ((12, 4096, 48, 205), 11), ((16, 4096, 32, 205), 11), ((10, 5120, 32, 256), 9)])
def test_lines_of_several_rounds(ask, shape, fewer):
    n, L, k, keep = shape
    on, off, short = ask([shape, (n, L, k, keep - 1), (fewer, L, k, keep)])
    assert on[1] >= min(L, 16 * keep) and off[1] == 0 and short[1] == 0


# where the union is slower by itself than the rows and one launch does not make up for it, (N, L, k, keep): eight wavefronts per tile of a
# short head, a second round that is mostly empty, one workgroup per CU
@pytest.mark.parametrize("shape", [(7, 640, 32, 128), (6, 768, 32, 154), (5, 900, 32, 180), (27, 640, 32, 80), (24, 700, 32, 88), (22, 768, 32, 96), (1, 12600, 32, 1050),
                                   (2, 13000, 32, 1084), (4, 14500, 32, 1209)])
def test_rows_where_they_are_faster(ask, shape):
    assert ask([shape])[0][1] == 0


def test_the_route_does_not_depend_on_the_projection(ask):
    """dsa_masked_attention has no use for k: the same lists give the same sums for every k."""
    shapes = [(n, L, keep) for n in (1, 2, 4, 7, 16, 64, 200) for L in (129, 250, 256, 300, 512, 640, 777, 1024, 1500, 2048, 3000, 4096, 5000, 6144, 8192, 9000, 12288, 16384)
              for keep in (1, L // 40, L // 21, L // 20, L // 12, L // 10, L // 8, L // 4, L // 2) if 1 <= keep <= 4096]
    answers = [ask([(n, L, k, keep) for n, L, keep in shapes]) for k in range(16, 129, 16)]
    taken = 0
    for shape, each in zip(shapes, zip(*answers)):
        assert len({a[1:] for a in each}) == 1, shape
        if each[0][1]:
            taken += 1
            assert len(set(each)) == 1, shape              # and the same wavefronts
    assert taken > 100


F32, BF16 = 0, 1


def test_two_tiles_at_5_to_10_percent(ask):
    """At k = 64 the predictor has two tiles of units per workgroup up to 10 %, from a round of wavefronts on, and for fp32 where the attention fits the launch."""
    def wavefronts(n, keep, dtype, d):
        return ask([(n, 4096, 64, keep, 0.125, dtype, d)])[0][0]
    for dtype, d in ((F32, 64), (F32, 128), (BF16, 128), (BF16, 64)):
        assert wavefronts(3, 205, dtype, d) == 0 and wavefronts(3, 206, dtype, d) > 0 and wavefronts(4, 206, dtype, d) == 0
    for dtype, d in ((F32, 64), (F32, 128)):
        assert wavefronts(4, 384, dtype, d) == 0 and wavefronts(4, 385, dtype, d) > 0
    assert wavefronts(4, 409, BF16, 128) == 0


def test_one_tile_for_the_sake_of_the_union(ask):
    """A shape that would have two tiles of units per workgroup if it were of d = 128, whose rows know no union, has one only if it takes the union."""
    shapes = [(n, L, keep) for n in (1, 2, 3, 4, 5, 8, 12, 16, 64) for L in (2048, 3584, 4096, 5120, 6144, 7168, 8192, 12288, 16384)
              for keep in range(L // 25, L // 8, 13)]
    narrow, wide = (ask([(n, L, 64, keep, 0.125, BF16, d) for n, L, keep in shapes]) for d in (64, 128))
    ones = 0
    for shape, (W, most, _), (W128, _, _) in zip(shapes, narrow, wide):
        if W128 == 0 and W:
            assert most > 0, shape
            ones += 1
    assert ones > 100
