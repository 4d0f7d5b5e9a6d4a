"""The forward call where the launch that makes the lists also attends over them, on both sides of the line where it does: list
lengths around the gathers of the row loops (8, 4, 4 and 2 keys per load instruction for bf16 and fp32 at d = 64 and 128, four in
flight), row counts that leave a workgroup with one unit, groups of rows.  The result has to be that of the two entry points one
after the other, bit for bit, and the oracle's within the bounds that the other tests use.  Which of the two routes a call took is
told by the number of kernels that it leaves in a captured graph, and every case says which one it stands for."""
import ctypes

import numpy as np
import pytest

import dsa_inputs as di

pytestmark = pytest.mark.gpu
TOL = {"f32": 1e-4, "bf16": 2e-2}


@pytest.fixture(scope="module")
def dsa():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("these tests need the MI355X: run them with -m gpu on the GPU box")
    import paper_2110_11299_amd as pkg
    pkg.binding.lib()
    return pkg


def captured_kernels(call):
    """Kernels that `call`, which allocates nothing, enqueues on the current stream: it is captured and not run."""
    import torch
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line)      # the runtime that torch loaded
    hip = ctypes.CDLL(path)
    stream = torch.cuda.Stream()
    graph, n = ctypes.c_void_p(), ctypes.c_size_t()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        assert hip.hipStreamBeginCapture(ctypes.c_void_p(stream.cuda_stream), 1) == 0
        try:
            call()
        finally:
            ended = hip.hipStreamEndCapture(ctypes.c_void_p(stream.cuda_stream), ctypes.byref(graph))
    assert ended == 0 and hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    nodes = (ctypes.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(graph, nodes, ctypes.byref(n)) == 0
    for node in nodes:
        kind = ctypes.c_int(-1)
        assert hip.hipGraphNodeGetType(ctypes.c_void_p(node), ctypes.byref(kind)) == 0 and kind.value == 0      # a kernel
    assert hip.hipGraphDestroy(graph) == 0
    return n.value


def forward(dsa, launches, dtype, H, L, d, vec, k, keep, scale=0.125, change=None):
    import torch
    print(f"[forward] {dtype} H={H} L={L} d={d} vec={vec} k={k} keep={keep} scale={scale}", flush=True)
    x = di.make_inputs(di.custom_config("fwd", B=1, H=H, L=L, d=d, dtype=dtype, rank=8, k=k, vec=vec, keep=keep, seed=L + keep))
    qkv = [np.array(a) for a in (x.Q, x.K, x.V)]
    if change:
        change(qkv)
    t, code = (torch.float32, dsa.DSA_F32) if dtype == "f32" else (torch.bfloat16, dsa.DSA_BF16)
    sh = dsa.make_shape(1, H, L, d, k, keep, vec, code, scale)
    dev = [torch.from_numpy(a).cuda().to(t) for a in qkv]
    codes = [torch.from_numpy(a).cuda() for a in (x.Qt, x.Kt)]
    O, idx = dsa.dsa_attention_fwd(sh, *dev, *codes)
    again, ws = (torch.empty_like(O), torch.empty_like(idx)), torch.empty(dsa.workspace_bytes(sh), dtype=torch.uint8, device="cuda")
    assert captured_kernels(lambda: dsa.dsa_attention_fwd(sh, *dev, *codes, O=again[0], idx_out=again[1], ws=ws)) == launches
    idx2 = dsa.dsa_predict_mask(sh, *codes)
    O2 = dsa.dsa_masked_attention(sh, *dev, idx2)
    assert torch.equal(idx, idx2)
    assert torch.equal(O.view(torch.int32), O2.view(torch.int32))
    return qkv, idx.cpu().numpy().reshape(-1, keep), O.cpu().numpy().reshape(-1, d)


def check(dsa, oracle, launches, dtype, H, L, d, vec, k, keep, scale=0.125):
    qkv, idx, got = forward(dsa, launches, dtype, H, L, d, vec, k, keep, scale)
    want = oracle.masked_attention(*qkv, idx, scale, vec).reshape(-1, d)
    assert np.abs(got - want).max() <= TOL[dtype]


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 128), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("keep", [1, 2, 4, 5, 8, 9, 15, 16, 17, 24, 25, 32, 33, 47, 65, 97])
def test_list_lengths(dsa, oracle, dtype, d, keep):
    check(dsa, oracle, 1, dtype, 80, 97, d, 1, 16, keep, scale=0.125 if keep % 2 else -0.125)


# few workgroups and short or long lists; groups of rows with places of the chip left idle, and without; more than four units to a
# wavefront; two tiles of units per workgroup; a list that leaves a CU one workgroup; ranges of several groups with a ragged end
@pytest.mark.parametrize("launches,dtype,H,L,d,vec,k,keep", [
    (1, "f32", 2, 256, 64, 1, 16, 4), (2, "f32", 2, 256, 64, 1, 16, 26), (1, "bf16", 1, 1000, 64, 1, 32, 10), (2, "bf16", 1, 1000, 64, 1, 32, 200),
    (2, "f32", 130, 200, 64, 4, 32, 20), (2, "f32", 140, 136, 128, 8, 32, 14), (2, "f32", 2, 1000, 64, 8, 16, 100), (2, "bf16", 130, 200, 64, 8, 32, 20),
    (2, "bf16", 130, 520, 64, 4, 32, 52), (2, "bf16", 140, 264, 64, 8, 16, 33), (2, "bf16", 17, 4104, 64, 8, 64, 205), (2, "bf16", 9, 8200, 64, 8, 64, 410),
    (1, "bf16", 4, 4100, 64, 1, 64, 60), (1, "bf16", 4, 4090, 64, 1, 64, 60), (1, "f32", 3, 8150, 128, 1, 64, 100), (1, "bf16", 3, 4096, 64, 1, 32, 410), (2, "bf16", 2, 4096, 128, 1, 48, 1300), (1, "bf16", 16, 777, 128, 1, 96, 39),
    (1, "f32", 20, 513, 128, 1, 128, 51), (1, "bf16", 2, 8200, 64, 1, 32, 82),
    (2, "f32", 60, 552, 128, 8, 32, 39), (2, "f32", 8, 4448, 64, 8, 32, 94), (2, "f32", 113, 1216, 64, 8, 16, 17), (1, "f32", 65, 692, 64, 4, 32, 7),
    (1, "f32", 127, 952, 64, 8, 64, 17), (2, "bf16", 108, 264, 64, 4, 16, 14), (2, "bf16", 103, 664, 64, 4, 48, 40), (1, "bf16", 29, 2128, 64, 4, 64, 62)])
def test_shapes(dsa, oracle, launches, dtype, H, L, d, vec, k, keep):
    check(dsa, oracle, launches, dtype, H, L, d, vec, k, keep)


# units of several rows in the kernels of every range length: fp32 of both widths, bf16, 9 to 16 groups per range (four and eight
# wavefronts), two tiles of units per workgroup
# two tiles of units per workgroup with lists of 5 to 10 % (k = 64): the longest that fp32 rows have in one launch, one key more, 8 % at d = 128, less than a round
@pytest.mark.parametrize("launches,dtype,H,d,keep", [(1, "f32", 4, 64, 384), (1, "f32", 4, 128, 384), (1, "f32", 4, 64, 385), (1, "bf16", 4, 128, 330), (1, "bf16", 4, 64, 250),
                                                     (1, "f32", 3, 64, 206), (1, "bf16", 3, 64, 380)])
def test_two_tiles(dsa, oracle, launches, dtype, H, d, keep):
    check(dsa, oracle, launches, dtype, H, 4096, d, 1, 64, keep)


@pytest.mark.parametrize("dtype,H,L,d,vec,k,keep", [
    ("f32", 250, 504, 64, 8, 32, 20), ("f32", 256, 512, 128, 8, 32, 20), ("f32", 64, 2044, 128, 4, 16, 40), ("f32", 32, 4088, 64, 8, 16, 40),
    ("f32", 16, 8184, 128, 4, 32, 80), ("f32", 4, 16376, 64, 8, 32, 160), ("f32", 16, 8192, 128, 8, 64, 80), ("bf16", 64, 2004, 64, 4, 16, 150),
    ("bf16", 64, 2000, 64, 8, 32, 60), ("bf16", 25, 5112, 64, 8, 32, 100), ("bf16", 32, 8184, 64, 8, 32, 80), ("bf16", 7, 8264, 64, 8, 32, 80),
    ("bf16", 7, 8264, 64, 8, 16, 80), ("bf16", 30, 4104, 64, 8, 48, 100), ("bf16", 6, 5000, 64, 4, 112, 100), ("bf16", 4, 16376, 64, 8, 128, 120),
    ("bf16", 16, 8192, 64, 8, 64, 80)])
def test_groups_in_one_launch(dsa, oracle, dtype, H, L, d, vec, k, keep):
    check(dsa, oracle, 1, dtype, H, L, d, vec, k, keep)


@pytest.mark.parametrize("vec", [4, 8])
def test_large_values_in_groups(dsa, oracle, vec):
    """Units whose sums leave fp32 on the first round (weights of up to 2^16, values of 2^118): done again within the same launch."""
    def change(qkv):
        qkv[0][...] *= 8.0
        qkv[2][...] = np.where(qkv[2] > 0, 2.0 ** 119, 2.0 ** 118)
    qkv, idx, got = forward(dsa, 1, "bf16", {4: 100, 8: 200}[vec], 520, 64, vec, 32, 75, scale=1.0, change=change)
    want = oracle.masked_attention(*qkv, idx, 1.0, vec).reshape(-1, 64)
    assert np.abs(got / want - 1.0).max() <= 2.0 ** -12      # weights 2^-16; scores of up to 2^9 in fp32 on either side


@pytest.mark.parametrize("d,keep", [(64, 24), (64, 28), (128, 22), (128, 30)])
def test_infinite_value_at_the_end_of_a_list(dsa, oracle, d, keep):
    """Lists that are a whole number of load instructions: no entry beyond the list makes NaN of an infinite value."""
    def change(qkv):
        qkv[2][0, :, -30:, 5] = np.inf
    qkv, idx, got = forward(dsa, 1, "f32", 80, 97, d, 1, 16, keep, change=change)
    want = oracle.masked_attention(*qkv, idx, 0.125, 1).reshape(-1, d)
    ok = np.isfinite(want)
    assert 0 < (~ok).sum() < want.size and not np.isnan(want).any()
    assert np.array_equal(got[~ok], want[~ok])
    assert np.abs(got[ok] - want[ok]).max() <= TOL["f32"]


@pytest.mark.parametrize("d,keep", [(64, 1), (64, 25), (64, 27), (128, 23), (128, 31)])
def test_infinite_value_inside_a_load(dsa, oracle, d, keep):
    """Lists that end inside a load instruction: the lanes behind the end add nothing, in the forward, from ELL and from CSR lists.
    (fp32: in bf16 a row's products pair a weight with a zero, which an infinite value in the neighbouring column makes NaN.)"""
    import torch

    def change(qkv):
        qkv[2][0, :, -30:, 5] = np.inf
    qkv, idx, got = forward(dsa, 1, "f32", 80, 97, d, 1, 16, keep, change=change)
    want = oracle.masked_attention(*qkv, idx, 0.125, 1).reshape(-1, d)
    sh = dsa.make_shape(1, 80, 97, d, 16, keep, 1, dsa.DSA_F32, 0.125)
    dev = [torch.from_numpy(a).cuda() for a in qkv]
    lists = torch.from_numpy(np.ascontiguousarray(idx)).cuda()
    csr = dsa.dsa_masked_attention_csr(sh, *dev, torch.arange(80 * 97 + 1, device="cuda", dtype=torch.int32) * keep, lists.flatten())
    S = dsa.dsa_sddmm(sh, *dev[:2], lists.view(1, 80, 97, keep))
    staged = dsa.dsa_spmm(sh, dsa.dsa_sparse_softmax(sh, S), lists.view(1, 80, 97, keep), dev[2])
    ok = np.isfinite(want)
    assert 0 < (~ok).sum() < want.size and not np.isnan(want).any()
    for out in (got, csr.cpu().numpy().reshape(-1, d), staged.cpu().numpy().reshape(-1, d)):
        assert np.array_equal(out[~ok], want[~ok])
        assert np.abs(out[ok] - want[ok]).max() <= TOL["f32"]


@pytest.mark.parametrize("bits", [8, 4])
def test_output_over_the_codes(dsa, bits):
    """Codes (or, packed, the workspace that they are widened in) in the memory that becomes the output: two launches, since the codes
    of a head are read by all of its workgroups."""
    import torch
    H, L, d, k, keep = 64, 513, 64, 32, 20
    gen = torch.Generator(device="cuda")
    gen.manual_seed(bits)
    Q, K, V = (torch.randn((1, H, L, d), generator=gen, device="cuda") for _ in range(3))
    top = 2 ** (bits - 1)
    Qt, Kt = (torch.randint(1 - top, top, (1, H, L, k), generator=gen, device="cuda", dtype=torch.int8) for _ in range(2))
    sh = dsa.make_shape(1, H, L, d, k, keep, 1, dsa.DSA_F32, 0.125)
    idx = torch.empty((1, H, L, keep), dtype=torch.int32, device="cuda")
    memory = torch.zeros(H * L * d, dtype=torch.float32, device="cuda")
    O, raw = memory.view(1, H, L, d), memory.view(torch.int8)
    if bits == 8:
        over = [raw[i * H * L * k:][:H * L * k].view(1, H, L, k) for i in range(2)]
        ws = torch.empty(dsa.workspace_bytes(sh), dtype=torch.uint8, device="cuda")
        want = [x.clone() for x in dsa.dsa_attention_fwd(sh, Q, K, V, Qt, Kt)]
        apart = lambda: dsa.dsa_attention_fwd(sh, Q, K, V, Qt, Kt, O=O, idx_out=idx, ws=ws)  # noqa: E731
        call = lambda: dsa.dsa_attention_fwd(sh, Q, K, V, *over, O=O, idx_out=idx, ws=ws)  # noqa: E731
        launches = (1, 2)
    else:
        packed = [((x[..., ::2] & 15) | (x[..., 1::2] << 4)).view(torch.uint8).contiguous() for x in (Qt, Kt)]
        ws = torch.empty(dsa.binding.workspace_bytes_bits(sh, bits), dtype=torch.uint8, device="cuda")
        want = [x.clone() for x in dsa.dsa_attention_fwd_bits(sh, bits, Q, K, V, *packed)]
        apart = lambda: dsa.dsa_attention_fwd_bits(sh, bits, Q, K, V, *packed, O=O, idx_out=idx, ws=ws)  # noqa: E731
        call = lambda: dsa.dsa_attention_fwd_bits(sh, bits, Q, K, V, *packed, O=O, idx_out=idx, ws=memory.view(torch.uint8))  # noqa: E731
        launches = (2, 3)             # one for the packed codes
    print(f"[over] bits={bits}", flush=True)
    assert captured_kernels(apart) == launches[0] and captured_kernels(call) == launches[1]
    if bits == 8:
        for place, codes in zip(over, (Qt, Kt)):
            place.copy_(codes)
    call()
    torch.cuda.synchronize()
    assert torch.equal(idx, want[1].view_as(idx)) and torch.equal(O, want[0])
