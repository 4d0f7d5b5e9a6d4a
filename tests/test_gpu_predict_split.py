"""The key-splitting mask predictor at the sizes where its plan changes (one key group per lane range, odd numbers of
groups, 1 to 16 wavefronts), at the edges of keep, and on score orders for which its first guess of the threshold
bracket is wrong, so that it has to sweep again.  Masks are whole numbers: every one is compared exactly."""
import numpy as np
import pytest

import dsa_inputs as di
from test_split_window_host import codes_of

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dsa():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("these tests need the MI355X: run them with -m gpu on the GPU box")
    import paper_2110_11299_amd as pkg
    pkg.binding.lib()
    return pkg


def check(dsa, oracle, Qt, Kt, keep, vec, label):
    import torch
    B, H, L, k = Qt.shape
    print(f"[split] {label} B={B} H={H} L={L} k={k} vec={vec} keep={keep}", flush=True)
    sh = dsa.make_shape(B, H, L, 64, k, keep, vec, dsa.DSA_F32, 0.125)
    got = dsa.dsa_predict_mask(sh, torch.from_numpy(Qt).cuda(), torch.from_numpy(Kt).cuda()).cpu().numpy().reshape(-1, keep)
    units = np.unique(np.linspace(0, got.shape[0] - 1, min(got.shape[0], max(32, (1 << 24) // L)), dtype=np.int64))
    want = oracle.predict_mask(Qt, Kt, keep, vec, units=units)
    bad = int((got[units] != want).any(axis=1).sum())
    assert bad == 0, f"{bad} of {len(units)} units differ"
    assert (np.diff(got, axis=1) > 0).all() and got.min() >= 0 and got.max() < L


# one key group per range (1, 2, 4, 8 wavefronts), one key more; 3 groups; 8 and 16 groups, a ragged last range
@pytest.mark.parametrize("L", [127, 128, 129, 256, 257, 511, 512, 513, 1025, 1537, 4095, 4097, 8193, 16385])
@pytest.mark.parametrize("k", [16, 32, 48, 64, 96])
def test_lengths(dsa, oracle, L, k):
    Qt, Kt = di.random_int8_case(L + k, 1, 2, L, k)
    check(dsa, oracle, Qt, Kt, max(1, L // 20), 1, "length")
    for vec in (4, 8):
        Lv = L // vec * vec
        check(dsa, oracle, np.ascontiguousarray(Qt[:, :, :Lv]), np.ascontiguousarray(Kt[:, :, :Lv]), max(1, Lv // 33), vec, "length")


@pytest.mark.parametrize("L", [96, 512, 1600, 4096, 9000])
def test_keep_edges(dsa, oracle, L):
    Qt, Kt = di.random_int8_case(L, 1, 1, L, 32)
    for keep in sorted({1, 2, 15, 16, 17, L // 3, L // 2, L - 1, L}):
        check(dsa, oracle, Qt, Kt, keep, 1, "keep")


@pytest.mark.parametrize("L,keep", [(700, 60), (4096, 205), (4096, 1500), (12000, 120)])
def test_score_orders(dsa, oracle, L, keep):
    """Scores that rise or fall with the key (the largest ones fill few buckets), a block of large ones, two values
    per key parity, and one outlier far above the rest (the histogram's range)."""
    k = 32
    pos = np.arange(L)
    orders = {
        "rising": pos * 254 // L - 127,
        "falling": 127 - pos * 254 // L,
        "block": np.where((pos > L // 2) & (pos < L // 2 + 2 * keep), 100, -20),
        "parity": np.where(pos % 2 == 0, 3, -3),
        "outlier": np.where(pos == L // 3, 127, (pos * 7919) % 5),
    }
    rng = np.random.Generator(np.random.Philox(L + keep))
    for name, v in orders.items():
        Kt = np.zeros((1, 1, L, k), np.int8)
        Kt[..., 0] = v
        Kt[..., 1] = rng.integers(-2, 3, size=L)
        Qt = np.zeros((1, 1, L, k), np.int8)
        Qt[..., 0] = np.where(pos % 3 == 0, 127, np.where(pos % 3 == 1, -127, 1))
        Qt[..., 1] = rng.integers(-1, 2, size=L)
        for vec in (1, 8):
            Lv = L // vec * vec
            check(dsa, oracle, np.ascontiguousarray(Qt[:, :, :Lv]), np.ascontiguousarray(Kt[:, :, :Lv]), keep, vec, name)


# where a threshold and a score are as far apart as they get: a group of 8 rows at k = 64 has scores from -8 * 64 * 16256 to 8 * 64 * 16384, and the
# signs of differences are taken from eight bits that are copies of it below 2^24 only (k = 128: from the sign itself)
@pytest.mark.parametrize("L", [520, 1040, 4104])
@pytest.mark.parametrize("k,vec", [(16, 1), (32, 8), (48, 8), (64, 1), (64, 4), (64, 8), (128, 8)])
def test_extreme_codes(dsa, oracle, L, k, vec):
    rng = np.random.Generator(np.random.Philox(L + k + vec))
    Qt = np.full((1, 2, L, k), -128, np.int8)
    Qt[:, 1] = rng.integers(-128, 128, size=(L, k))
    Qt[:, :, ::24] = 127
    Kt = np.where(rng.random((1, 2, L, 1)) < 0.5, -128, 127).astype(np.int8) * np.ones((1, 1, 1, k), np.int8)
    Kt[:, :, 5::7] = rng.integers(-128, 128, size=Kt[:, :, 5::7].shape)
    Kt[:, :, 3::11, : k // 2] = 127
    for keep in (1, L // 50, L // 12, L // 2, L - 3):
        check(dsa, oracle, Qt, np.ascontiguousarray(Kt), keep, vec, "extreme")


# heads that end inside a lane range, whose buckets have fewer keys than the others (the masks; that the thresholds do not follow such buckets, which would
# cost sweeps, is asked in test_split_window_host.py, at lengths like these)
@pytest.mark.parametrize("L,k,vec,keep", [(2104, 32, 1, 32), (3680, 16, 1, 40), (7792, 32, 8, 145), (896, 32, 1, 36), (1032, 64, 1, 20)])
def test_ragged_ranges(dsa, oracle, L, k, vec, keep):
    x = di.make_inputs(di.custom_config("ragged", B=1, H=2, L=L, d=64, dtype="bf16", rank=32, k=k, vec=vec, keep=keep, seed=L))
    check(dsa, oracle, x.Qt, x.Kt, keep, vec, "ragged")


# thresholds that the first histogram does not have, below it and above it: in every kernel with a second one (2 to 16 words per lane, one tile and two, ranges
# that end beyond the head) and in those without (one word; groups at k = 16)
@pytest.mark.parametrize("H,L,vec,k,keep", [
    (2, 500, 1, 32, 50), (2, 504, 8, 16, 30), (4, 1600, 1, 16, 90), (4, 1604, 4, 16, 90), (4, 1600, 8, 32, 90), (2, 2104, 1, 48, 32), (2, 2048, 8, 64, 102), (2, 2050, 1, 112, 100),
    (2, 2048, 4, 128, 60), (4, 4096, 1, 32, 410), (4, 4104, 8, 48, 205), (2, 4096, 1, 64, 82), (1, 4500, 1, 96, 220), (2, 8192, 1, 32, 410), (1, 8200, 8, 64, 400), (1, 12000, 1, 16, 120),
    (16, 8192, 8, 64, 82), (1, 16384, 1, 64, 164), (1, 16384, 8, 128, 164)])
def test_thresholds_outside_of_the_window(dsa, oracle, H, L, vec, k, keep):
    rng = np.random.Generator(np.random.Philox(L + keep + k))
    for kind in ("5 %", "log-normal", "clusters", "sinks"):
        Qt, Kt = (np.stack(x)[None].astype(np.int8) for x in zip(*[codes_of(rng, L, k, kind, L) for _ in range(H)]))
        check(dsa, oracle, Qt, Kt, keep, vec, kind)


# the same orders in every kernel: all projection dimensions, 1, 4, 8 and 16 groups per range with one tile, 4 and 8 with two
@pytest.mark.parametrize("H,L,vec,k,keep", [
    (2, 512, 1, 16, 30), (2, 512, 8, 48, 30), (2, 512, 1, 128, 30), (2, 1600, 1, 48, 90), (2, 1600, 4, 64, 90), (2, 1600, 8, 96, 90),
    (4, 4096, 1, 16, 205), (5, 4096, 1, 32, 205), (5, 4096, 8, 64, 205), (5, 4096, 1, 112, 205), (1, 12000, 1, 64, 600), (1, 12000, 4, 16, 120),
    (1, 12000, 8, 128, 120), (16, 2050, 1, 64, 60), (2, 4100, 1, 48, 80), (1, 16384, 1, 64, 500), (16, 8192, 8, 64, 250),
    (3, 4040, 1, 64, 60), (2, 6100, 1, 64, 60), (2, 8100, 1, 48, 80), (16, 8072, 8, 64, 250)])
def test_score_orders_in_every_kernel(dsa, oracle, H, L, vec, k, keep):
    """As above, and tiles of 16 units that need no second sweep next to tiles that do (of a workgroup with two tiles one is good
    while the other is swept again)."""
    pos = np.arange(L)
    orders = {
        "rising": pos * 254 // L - 127,
        "block": np.where((pos > L // 2) & (pos < L // 2 + 2 * keep), 100, -20),
        "parity": np.where(pos % 2 == 0, 3, -3),
        "outlier": np.where(pos == L // 3, 127, (pos * 7919) % 5),
    }
    rng = np.random.Generator(np.random.Philox(L + keep + k))
    for name, v in orders.items():
        Kt = np.zeros((1, H, L, k), np.int8)
        Kt[..., 0] = v
        Kt[..., 1] = rng.integers(-2, 3, size=L)
        Kt[..., k - 2] = rng.integers(-127, 128, size=(1, H, L))          # what the even tiles see, and nothing else
        tile = pos // (16 * vec) % 2
        Qt = np.zeros((1, H, L, k), np.int8)
        Qt[..., 0] = tile * np.where(pos // vec % 3 == 0, 127, np.where(pos // vec % 3 == 1, -127, 1))
        Qt[..., 1] = tile * rng.integers(-1, 2, size=L)
        Qt[..., k - 2] = (1 - tile) * rng.integers(1, 100, size=(1, H, L))
        check(dsa, oracle, Qt, Kt, keep, vec, name)


# ranges of one group, whose bands are scored two slots at a time up to 32 keys and four beyond, with an order by counting up to 16: bands of
# few keys, of a bin or two, and of whole plateaus (codes of few levels), in every kernel
@pytest.mark.parametrize("levels", [1, 3, 127])
@pytest.mark.parametrize("H,L,vec", [(4, 1024, 1), (5, 1000, 8), (3, 500, 1), (800, 128, 4)])
def test_bands_of_one_group(dsa, oracle, H, L, vec, levels):
    rng = np.random.Generator(np.random.Philox(L + levels))
    for k in (16, 32, 48, 64, 112, 128):
        Qt, Kt = (rng.integers(-levels, levels + 1, size=(1, H, L, k), dtype=np.int8) for _ in range(2))
        for keep in (L // 100 + 1, L // 10, L // 3):
            check(dsa, oracle, Qt, Kt, keep, vec, f"bands, {levels} levels,")


# two tiles of units per workgroup (projection dimensions of 48 and 64, enough units): a tile that is partly or wholly
# beyond the head, ranges of 2, 3 and 8 groups, keep at the edge of what its 16 buckets per lane take
@pytest.mark.parametrize("H,L,vec", [(16, 1025, 1), (15, 1100, 1), (60, 1104, 4), (8, 2049, 1), (30, 8200, 8)])
@pytest.mark.parametrize("k", [48, 64])
def test_pairs_of_tiles(dsa, oracle, H, L, vec, k):
    Qt, Kt = di.random_int8_case(L + H, 1, H, L, k)
    for keep in (1, 30, 409, 410):
        check(dsa, oracle, Qt, Kt, keep, vec, "pairs")


# the same where the plan takes two tiles now, and on both sides of its lines: ranges that end at the head, 1 to 1/64 of it beyond and
# farther, four and five words, half a round of wavefronts, two rounds, the longest list, the two lengths that differ in wavefronts
@pytest.mark.parametrize("H,L,vec,k,keep", [(2, 4100, 1, 64, 409), (2, 4100, 1, 48, 82), (16, 2050, 1, 64, 64), (1, 16384, 1, 64, 512),
                                            (1, 16384, 1, 48, 327), (16, 8192, 8, 64, 256), (8, 8200, 4, 64, 256), (16, 8192, 8, 64, 257),
                                            (4, 4100, 1, 64, 409), (64, 1040, 1, 64, 10), (16, 8192, 8, 48, 82),
                                            (2, 4096, 1, 64, 205), (2, 4095, 1, 64, 1), (3, 4033, 1, 64, 200), (3, 4032, 1, 64, 200), (2, 5041, 1, 64, 253), (2, 5042, 1, 64, 253),
                                            (4, 4096, 1, 64, 206), (4, 4096, 1, 64, 384), (5, 4040, 1, 64, 300), (4, 5110, 1, 64, 384), (4, 4096, 1, 64, 385), (3, 4096, 1, 64, 206),
                                            (1, 8192, 1, 64, 409), (1, 8066, 1, 48, 400), (2, 16133, 1, 64, 512), (2, 16161, 1, 48, 160),
                                            (17, 8064, 8, 64, 252), (17, 8072, 8, 64, 1), (9, 12280, 8, 64, 300), (5, 16136, 4, 64, 500)])
def test_pairs_of_tiles_in_the_plan(dsa, oracle, H, L, vec, k, keep):
    Qt, Kt = di.random_int8_case(L + H + keep, 1, H, L, k)
    check(dsa, oracle, Qt, Kt, keep, vec, "pairs in the plan")


@pytest.mark.parametrize("H,L", [(256, 128), (257, 128), (48, 256), (49, 256), (1, 2047), (1, 2048), (3, 4096), (4, 4096), (1, 8192), (2, 8192)])
def test_wavefronts_of_the_plan(dsa, oracle, H, L):
    for k in (32, 96):
        Qt, Kt = di.random_int8_case(L + H, 1, H, L, k)
        check(dsa, oracle, Qt, Kt, max(1, L // 40), 1, "wavefronts")


# two contraction steps: 112 (the second one partly empty) and 128 (its halves of odd rows change places), in every number of
# groups per range that has a kernel of its own
@pytest.mark.parametrize("H,L", [(2, 130), (2, 1025), (4, 4096), (1, 8193), (1, 16385)])
@pytest.mark.parametrize("k", [112, 128])
def test_two_steps(dsa, oracle, H, L, k):
    Qt, Kt = di.random_int8_case(L + k, 1, H, L, k)
    for vec in (1, 4, 8):
        Lv = L // vec * vec
        check(dsa, oracle, np.ascontiguousarray(Qt[:, :, :Lv]), np.ascontiguousarray(Kt[:, :, :Lv]), max(1, L // 50), vec, "two steps")


# heads shorter than what a lane range's later batches of key rows start at (28 rows), where every one of them lies beyond the head
@pytest.mark.parametrize("k", [16, 48, 64, 80, 112, 128])
def test_short_heads(dsa, oracle, k):
    for L in (1, 2, 3, 7, 8, 12, 15, 16, 17, 23, 24, 27, 28, 31, 32):
        Qt, Kt = di.random_int8_case(L + k, 1, 3, L, k)
        for vec in (1, 4, 8):
            if L % vec == 0:
                for keep in sorted({1, (L + 1) // 2, L}):
                    check(dsa, oracle, Qt, Kt, keep, vec, "short")
