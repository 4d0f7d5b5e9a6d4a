"""The addresses of the predictor's key loads, counted out on the CPU from the functions that the kernel takes them from
(csrc/key_rows.h).  The range check of a buffer load is taken as what every description of it agrees on: a request whose vector
and immediate offset reach the descriptor's length gives zeros, and nothing is said about the scalar offset, which therefore has
to be zero (asserted on the kernel's source)."""
import re
import subprocess
from pathlib import Path

CSRC = Path(__file__).resolve().parent.parent / "paper_2110_11299_amd" / "csrc"

PROGRAM = r"""
#include "key_rows.h"
#include <cstdio>
#include <cstdlib>
#include <vector>
using namespace dsa;

// every request of a workgroup of W wavefronts
static void check(int k, int L, int W, bool half)
{
    const int NW = (L + 128 * W - 1) / (128 * W), Lr = 32 * NW;
    const int R = k == 16 ? 4 : k == 32 ? 2 : 1, STEPS = k <= 64 ? 1 : 2, NS = 8 / R;
    const int NSB = key_batch_slots(NS, STEPS, half), BPG = NS / NSB, batches = NW * BPG, step = key_slot_step(k, R);
    const bool constant = k == 16 || k == 32 || k == 48 || k == 64 || k == 128;
    std::vector<char> seen((size_t)L * (k / 16), 0);
    for (int wv = 0; wv < W; ++wv)
        for (int lane = 0; lane < 64; ++lane) {
            const unsigned row0 = key_row_offset(wv, lane, Lr, k, R);
            for (int b = 0; b <= batches; ++b)
                for (int sl = 0; sl < NSB; ++sl)
                    for (int s = 0; s < STEPS; ++s)
                        for (int twist = 0; twist <= (k == 64); ++twist) {
                            const int piece = key_piece_offset(lane, k, R, s);
                            const unsigned at = row0 + ((unsigned)(piece < 0 ? 0 : piece) ^ (twist && (lane & 2) ? 32u : 0u));
                            const int from = key_batch_offset(b, batches, NSB, step) + (constant ? 0 : sl * step);
                            const unsigned offset = at + (constant ? sl * step : 0);
                            const unsigned length = (unsigned)key_bytes_left(L, k, from);
                            if (offset >= length) continue;                                // zeros
                            const long long byte = (long long)from + offset;
                            if (from < 0 || byte + 16 > (long long)L * k || offset + 16 > length || byte % 16) {
                                printf("k=%d L=%d W=%d wv=%d lane=%d b=%d sl=%d: byte %lld of %d\n", k, L, W, wv, lane, b, sl, byte, L * k);
                                exit(1);
                            }
                            // the piece of the row that the lane answers for
                            const int c = lane & 15, g = lane >> 4, tile = (b < batches ? b : batches - 1) * NSB + sl;
                            const int key = (4 * wv + (c >> 2)) * Lr + 4 * (tile * R + (R == 4 ? g : R == 2 ? g >> 1 : 0)) + (c & 3);
                            if (byte / k != key) { printf("k=%d L=%d W=%d: key %lld instead of %d\n", k, L, W, byte / k, key); exit(1); }
                            if (!twist && piece >= 0) seen[(size_t)(byte / 16)] = 1;
                        }
        }
    for (char x : seen)
        if (!x) { printf("k=%d L=%d W=%d: a piece of K~ is never fetched\n", k, L, W); exit(1); }
}

int main()
{
    for (int k = 16; k <= 128; k += 16)
        for (bool half : {false, true}) {
            for (int W : {1, 2, 4, 8, 16}) {
                for (int L = 1; L <= 132; ++L) check(k, L, W, half);
                for (int L : {255, 256, 257, 511, 513, 777, 2000, 2049, 4100}) check(k, L, W, half);
            }
            check(k, 8199, 8, half);
            for (int L : {16384, 16385, 32767, 32768}) check(k, L, 16, half);
        }
    puts("ok");
}
"""


def test_every_request_lies_inside_the_head(tmp_path):
    src, exe = tmp_path / "rows.cpp", tmp_path / "rows"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", f"-I{CSRC}", str(src), "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True)
    assert res.returncode == 0 and res.stdout.strip() == "ok", res.stdout


def test_no_scalar_offset():
    loads = re.findall(r"raw_buffer_load_\w+\((.*)\);", (CSRC / "predict_split.h").read_text())
    assert loads and all(re.search(r", 0, 0\)+$", a) for a in loads), loads
