"""Fused attention of vector-wise units (8 or 4 rows share a list, bfloat16) at the edges of its steps of 32 keys and of its
workgroups of four units, up to the longest list, with scores that outgrow its running reference, and with scales of any
sign.  Against the oracle on the same bf16 values, with the bound for bf16 inputs that the other tests use, and a two-norm bound
that tells the kernel's weights (two bf16, off by up to 2^-16 each, 2e-6 to 5e-6 together) from weights of one bf16 (2^-8,
4e-4 to 1.5e-3 together)."""
import numpy as np
import pytest

import dsa_inputs as di

pytestmark = pytest.mark.gpu
TOL = 2e-2
TWO_NORM = 5e-5         # 3.3 * 2^-16: the largest error of a weight, and one of fp32 exponentials and sums beside it


@pytest.fixture(scope="module")
def dsa():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("these tests need the MI355X: run them with -m gpu on the GPU box")
    import paper_2110_11299_amd as pkg
    pkg.binding.lib()
    return pkg


def case(H, L, d, vec, keep):
    x = di.make_inputs(di.custom_config("units", B=1, H=H, L=L, d=d, dtype="bf16", rank=8, k=16, vec=vec, keep=keep, seed=L + keep))
    rng = np.random.Generator(np.random.Philox(L + keep + vec))
    idx = np.stack([np.sort(rng.choice(L, keep, replace=False)) for _ in range(H * (L // vec))]).astype(np.int32)
    return [np.ascontiguousarray(a) for a in (x.Q, x.K, x.V)], idx


def run(dsa, qkv, idx, vec, scale):
    import torch
    _, H, L, d = qkv[0].shape
    keep = idx.shape[-1]
    print(f"[units] H={H} L={L} d={d} vec={vec} keep={keep} scale={scale}", flush=True)
    sh = dsa.make_shape(1, H, L, d, 16, keep, vec, dsa.DSA_BF16, scale)
    dev = [torch.from_numpy(a).cuda().bfloat16() for a in qkv]
    O = dsa.dsa_masked_attention(sh, *dev, torch.from_numpy(idx.reshape(1, H, L // vec, keep)).cuda())
    return O.cpu().numpy().reshape(-1, d)


def check(dsa, oracle, qkv, idx, vec, scale):
    want = oracle.masked_attention(*qkv, idx, scale, vec).reshape(-1, qkv[0].shape[-1])
    err = run(dsa, qkv, idx, vec, scale) - want
    print(f"    two-norm {np.linalg.norm(err) / np.linalg.norm(want):.2e}, largest {np.abs(err).max():.2e}", flush=True)
    assert np.abs(err).max() <= TOL
    assert np.linalg.norm(err) <= TWO_NORM * np.linalg.norm(want)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("vec", [4, 8])
@pytest.mark.parametrize("L,keep", [(8, 1), (40, 31), (40, 32), (72, 33), (136, 64), (264, 65), (264, 264), (1000, 97)])
def test_edges(dsa, oracle, d, vec, L, keep):
    qkv, idx = case(3, L, d, vec, keep)
    for scale in (0.125, -0.125, 0.0):
        check(dsa, oracle, qkv, idx, vec, scale)


@pytest.mark.parametrize("d,vec", [(64, 8), (128, 4)])
def test_longest_list(dsa, oracle, d, vec):
    qkv, _ = case(1, 64, d, vec, 1)
    L, keep = 4200, 4096
    rng = np.random.Generator(np.random.Philox(d))
    qkv = [np.ascontiguousarray(np.concatenate([a] * 66, axis=2)[:, :, :L]) for a in qkv]
    idx = np.stack([np.sort(rng.choice(L, keep, replace=False)) for _ in range(L // vec)]).astype(np.int32)
    check(dsa, oracle, qkv, idx, vec, 0.125)


@pytest.mark.parametrize("vec", [4, 8])
@pytest.mark.parametrize("order", [1, -1])
def test_scores_that_grow(dsa, oracle, vec, order):
    """Scores from 0 to 88, rising or falling along the list, in one query of the unit only."""
    qkv, idx = case(1, 640, 64, vec, 320)
    Q, K, _ = qkv
    Q[0, 0, ::vec] = 1.0
    K[...] = (np.arange(640)[::order] // 54).astype(np.float32)[None, None, :, None]
    check(dsa, oracle, qkv, idx, vec, 0.125)


@pytest.mark.parametrize("vec", [4, 8])
def test_scores_that_grow_within_the_slack(dsa, oracle, vec):
    """Scores that rise by 10.5 (2^15 between the weights) after the first step: the reference stays where it is, and the
    weights that count are thousands of times 1."""
    qkv, idx = case(1, 640, 64, vec, 320)
    Q, K, _ = qkv
    Q[...] = 0.0
    Q[0, 0, :, 0] = 1.0 + (np.arange(640) % 4) / 16.0
    K[...] = 0.0
    K[0, 0, :, 0] = np.round(np.arange(640) / 640 * 70.0)
    check(dsa, oracle, qkv, idx, vec, 0.125)


@pytest.mark.parametrize("vec", [4, 8])
def test_values_that_are_not_finite(dsa, oracle, vec):
    """They reach the rows that keep their key, with their sign, and no others."""
    qkv, idx = case(2, 600, 64, vec, 96)                # three whole steps
    V = qkv[2]
    V[0, 0, 5, 3], V[0, 0, 70, 7], V[0, 1, 590, 63], V[0, 1, 64, 0] = np.inf, np.nan, -np.inf, np.inf
    want = oracle.masked_attention(*qkv, idx, 0.125, vec).reshape(-1, 64)
    got = run(dsa, qkv, idx, vec, 0.125)
    ok = np.isfinite(want)
    assert 0 < (~ok).sum() < want.size
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(got[np.isinf(want)], want[np.isinf(want)])
    assert np.abs(got[ok] - want[ok]).max() <= TOL


@pytest.mark.parametrize("d,vec", [(64, 4), (64, 8), (128, 4), (128, 8)])
@pytest.mark.parametrize("keep", [1, 31, 33, 200])
def test_infinite_value_at_the_end_of_a_list(dsa, oracle, d, vec, keep):
    """The step of 32 keys that a list ends in is filled up with its last key: an infinite value there stays infinite."""
    qkv, idx = case(2, 600, d, vec, keep)
    V = qkv[2]
    V[0, 0, 599, 3], V[0, 1, 598, d - 1] = np.inf, -np.inf
    idx[::3, -1] = 599
    idx[1::3, -1] = 598
    idx[:, :-1] = np.minimum(idx[:, :-1], 597)              # (a key may then be listed twice: it counts twice)
    want = oracle.masked_attention(*qkv, idx, 0.125, vec).reshape(-1, d)
    got = run(dsa, qkv, idx, vec, 0.125)
    ok = np.isfinite(want)
    assert 0 < (~ok).sum() < want.size and not np.isnan(want).any()
    assert np.array_equal(got[~ok], want[~ok])
    assert np.abs(got[ok] - want[ok]).max() <= TOL


@pytest.mark.parametrize("d,vec", [(64, 4), (64, 8), (128, 4), (128, 8)])
@pytest.mark.parametrize("keep", [64, 75])
def test_large_values_with_scores_that_grow(dsa, oracle, d, vec, keep):
    """Scores that exceed those of the first 32 keys by 10 (a factor of 2^14.4 between the weights), values of 2^118 and
    2^119: sums of up to 75 of them with weights of at most 1 stay below 2^126.  Every value is positive, so the relative
    error is that of a weight (2^-16)."""
    qkv, idx = case(2, 320, d, vec, keep)
    Q, K, V = qkv
    Q[...], K[...] = 0.0, 0.0
    Q[..., 0] = 1.0
    K[:, :, 160:, 0] = 10.0
    V[...] = np.where(V > 0, 2.0 ** 119, 2.0 ** 118)
    idx[:, :32] = np.sort(idx[:, :32] % 160, axis=1)
    idx[:, 32:] = np.sort(160 + idx[:, 32:] % 160, axis=1)
    want = oracle.masked_attention(*qkv, idx, 1.0, vec).reshape(-1, d)
    got = run(dsa, qkv, idx, vec, 1.0)
    assert np.abs(got / want - 1.0).max() <= 2.0 ** -15
