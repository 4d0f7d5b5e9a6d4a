"""The work this library is called for, as cases that can be timed and compared.

Every case is one pass of Dynamic Sparse Attention over a [B, H, L, d] layer through the public entry points, with
Q, K, V (and, where the pass starts from them, the int8 projections) resident on the GPU, the workspace and the output
buffers kept by the caller, as the C ABI is meant to be used.  `op` says which entry points:

  fwd        dsa_attention_fwd on projections in hand (the call the headline rate is quoted on)
  layer      what a model's layer does with fresh Q, K, V: project and quantise Q and K, then the forward; with
             bits = 4 or 2 through the packed low-precision entry points
  threshold  a threshold mask in CSR form and the attention over it
  staged     the four stages one by one (mask, scores, softmax, output), scores and weights handed back

Inputs follow the repository's recipe (dsa_inputs.py): low-rank signal plus noise, a few high-norm "global" keys on
long sequences, one Gaussian projection shared by Q and K.
"""
import math

import torch

from paper_2110_11299_amd import binding as dsa


def _case(name, op, B, H, L, d, k, keep, vec, dtype, rank=32, n_global=0, bits=8):
    return {"name": name, "op": op, "B": B, "H": H, "L": L, "d": d, "k": k, "keep": keep, "vec": vec, "dtype": dtype,
            "rank": rank, "n_global": n_global, "bits": bits}


def listed():
    return [
        # one short sequence: two small launches, nothing but latency
        _case("tiny-fine", "fwd", 1, 2, 256, 64, 16, 26, 1, "f32", rank=8),
        # a BERT-base-shaped layer in fp32 at 10 %, a batch of 8, from fresh Q, K, V
        _case("base-fine", "layer", 8, 12, 512, 64, 32, 51, 1, "f32", rank=16),
        # vector-wise masks (8 query rows share a list) on a batch of medium sequences
        _case("medium-vec8", "fwd", 4, 16, 2048, 64, 32, 102, 8, "bf16"),
        # the headline shape: h = 8, l = 4096, d = 64 at 5 %, fine-grained and vector-wise
        _case("long-fine", "fwd", 2, 8, 4096, 64, 32, 205, 1, "bf16", n_global=16),
        _case("long-vec8", "fwd", 2, 8, 4096, 64, 32, 205, 8, "bf16", n_global=16),
        # the long stress shape at 1 %, wide heads
        _case("stress-vec8", "fwd", 1, 16, 8192, 128, 64, 82, 8, "bf16", rank=64, n_global=32),
        # INT4, the precision the method proposes for its predictor, from fresh Q, K, V
        _case("long-fine-int4", "layer", 2, 8, 4096, 64, 32, 205, 1, "bf16", n_global=16, bits=4),
        # the headline shape at 10 % (DSA-90): twice the list
        _case("long-fine-dense", "fwd", 2, 8, 4096, 64, 32, 410, 1, "bf16", n_global=16),
        # text classification: 4 heads, l = 2000, batch 16, 1x4 column vectors at 10 %; a length that is no
        # multiple of any tile
        _case("text-vec4", "layer", 16, 4, 2000, 64, 16, 200, 4, "bf16", n_global=8),
        # a tuned threshold instead of top-k: counts that differ from row to row
        _case("threshold-fine", "threshold", 2, 8, 2048, 64, 32, 102, 1, "bf16", n_global=8),
        # the longest sequences, fine-grained, at 1 %
        _case("longest-fine", "fwd", 1, 4, 16384, 128, 64, 164, 1, "bf16", rank=64, n_global=64),
        # the stages one by one on an odd length, wide heads, fp32
        _case("ragged-staged", "staged", 3, 5, 777, 128, 32, 39, 1, "f32", rank=16),
    ]


# Selections over keys and gathered bytes of the largest listed cases: a drawn case stays within one such budget.
_MOST_SCORES = 4 * 16384 * 16384
_MOST_GATHER = 2 * 2 * 8 * 4096 * 410 * 64 * 2


def draw(rng):
    while True:
        op = rng.choice(["fwd", "fwd", "fwd", "layer", "layer", "threshold", "staged"])
        vec = rng.choice([1, 1, 1, 4, 8, 8])
        L = int(round(math.exp(rng.uniform(math.log(96), math.log(16384)))))
        L = max(vec, L // vec * vec)
        N = int(round(math.exp(rng.uniform(0.0, math.log(192)))))
        H = next(h for h in (16, 12, 8, 5, 4, 3, 2, 1) if N % h == 0)
        d = rng.choice([64, 64, 128])
        k = rng.choice([16, 32, 32, 64] if op == "threshold" else [16, 32, 32, 32, 48, 64])
        ratio = math.exp(rng.uniform(math.log(0.01), math.log(0.12)))
        keep = dsa.keep_from_ratio(L, ratio)
        dtype = rng.choice(["bf16", "bf16", "f32"])
        bits = rng.choice([8, 8, 4, 2]) if op == "layer" else 8
        if op == "threshold" and N * L * L >= 1 << 29:
            continue
        e = 4 if dtype == "f32" else 2
        if N * (L // vec) * L / _MOST_SCORES + N * L * keep * d * e * 2 / _MOST_GATHER > 1.0:
            continue
        c = _case(None, op, N // H, H, L, d, k, keep, vec, dtype, rank=min(d // 2, rng.choice([8, 16, 32, 64])),
                  n_global=L // 256 if L >= 1024 and rng.random() < 0.7 else 0, bits=bits)
        del c["name"]
        return c


def _signal(gen, N, L, d, rank):
    u = torch.randn((N, L, rank), generator=gen, device="cuda")
    w = torch.randn((N, rank, d), generator=gen, device="cuda") * rank ** -0.5
    return torch.matmul(u, w) + 0.1 * torch.randn((N, L, d), generator=gen, device="cuda")


def _codes(x, R):
    y = x.double() @ R.double()
    return (y * (127.0 / y.abs().max())).round().clamp(-127, 127).to(torch.int8)


def prepare(case, seed):
    """Q, K, V, the projection or the codes, the workspace and the output buffers of one layer."""
    c = case
    B, H, L, d, k, vec, op = c["B"], c["H"], c["L"], c["d"], c["k"], c["vec"], c["op"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1000003 * int(seed) + 17)
    R = torch.randn((d, k), generator=gen, device="cuda") * k ** -0.5
    Q, K, V = (_signal(gen, B * H, L, d, c["rank"]) for _ in range(3))
    if c["n_global"]:
        # high-norm keys at positions drawn per head
        at = torch.rand((B * H, L), generator=gen, device="cuda").argsort(dim=1)[:, :c["n_global"]]
        K.scatter_(1, at[..., None].expand(-1, -1, d), 4.0 * K.gather(1, at[..., None].expand(-1, -1, d)))
    t = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    Q, K, V = (x.view(B, H, L, d).to(t).contiguous() for x in (Q, K, V))
    shape = dsa.make_shape(B, H, L, d, k, c["keep"], vec, dsa.DSA_F32 if c["dtype"] == "f32" else dsa.DSA_BF16, d ** -0.5)
    s = {"op": op, "shape": shape, "bits": c["bits"], "Q": Q, "K": K, "V": V,
         "O": torch.empty((B, H, L, d), dtype=torch.float32, device="cuda")}
    byte = lambda n: torch.empty(max(int(n), 16), dtype=torch.uint8, device="cuda")  # noqa: E731
    if op != "threshold":
        s["idx"] = torch.empty((B, H, L // vec, c["keep"]), dtype=torch.int32, device="cuda")
    if op == "layer":
        s["R"] = R.contiguous()
        s["project_ws"] = byte(dsa.project_workspace_bytes(shape))
        code = (B, H, L, k * c["bits"] // 8)
        kind = torch.int8 if c["bits"] == 8 else torch.uint8
        s["Qt"], s["Kt"] = (torch.empty(code, dtype=kind, device="cuda") for _ in range(2))
        s["ws"] = byte(dsa.workspace_bytes(shape) if c["bits"] == 8 else dsa.workspace_bytes_bits(shape, c["bits"]))
        return s
    s["Qt"], s["Kt"] = _codes(Q.float(), R), _codes(K.float(), R)
    if op == "threshold":
        # a threshold that about keep / L of the scores reach (tuned on every 37th unit), and a list with twice the
        # room: what lies behind the last row's keys stays zero
        q = s["Qt"].view(B * H, L // vec, vec, k).float().sum(2)
        kk = s["Kt"].view(B * H, L, k).float()
        some = torch.cat([torch.matmul(q[n, n % 37::37], kk[n].t()).flatten() for n in range(B * H)])
        theta = int(some.kthvalue(max(1, round((1.0 - c["keep"] / L) * some.numel()))).values.item())
        room = 2 * c["keep"] * B * H * (L // vec)
        while sum(int((torch.matmul(q[n], kk[n].t()) >= theta).sum(1).clamp(min=1).sum()) for n in range(B * H)) > room:
            theta += 1 + abs(theta) // 16
        s["theta"] = theta
        s["col"] = torch.zeros(room, dtype=torch.int32, device="cuda")
        s["row_ptr"] = torch.empty(B * H * (L // vec) + 1, dtype=torch.int32, device="cuda")
        s["ws"] = byte(dsa.threshold_workspace_bytes(shape))
    else:
        s["ws"] = byte(dsa.workspace_bytes(shape))
    if op == "staged":
        s["S"], s["P"] = (torch.empty((B, H, L, c["keep"]), dtype=torch.float32, device="cuda") for _ in range(2))
    return s


def run(s):
    """One pass; returns the output and the mask, and what else the entry points hand back."""
    sh, op = s["shape"], s["op"]
    if op == "fwd":
        return dsa.dsa_attention_fwd(sh, s["Q"], s["K"], s["V"], s["Qt"], s["Kt"], O=s["O"], idx_out=s["idx"], ws=s["ws"])
    if op == "layer":
        if s["bits"] == 8:
            for x, xt in (("Q", "Qt"), ("K", "Kt")):
                dsa.dsa_project_quantize(sh, s[x], s["R"], Xt=s[xt], ws=s["project_ws"], want_amax=False)
            O, idx = dsa.dsa_attention_fwd(sh, s["Q"], s["K"], s["V"], s["Qt"], s["Kt"], O=s["O"], idx_out=s["idx"], ws=s["ws"])
        else:
            for x, xt in (("Q", "Qt"), ("K", "Kt")):
                dsa.dsa_project_quantize_bits(sh, s["bits"], s[x], s["R"], Xt=s[xt], ws=s["project_ws"], want_amax=False)
            O, idx = dsa.dsa_attention_fwd_bits(sh, s["bits"], s["Q"], s["K"], s["V"], s["Qt"], s["Kt"], O=s["O"],
                                                idx_out=s["idx"], ws=s["ws"])
        return O, idx, s["Qt"], s["Kt"]
    if op == "threshold":
        row_ptr, col = dsa.dsa_predict_mask_threshold(sh, s["Qt"], s["Kt"], s["theta"], s["col"].numel(),
                                                      row_ptr=s["row_ptr"], col=s["col"], ws=s["ws"])
        return dsa.dsa_masked_attention_csr(sh, s["Q"], s["K"], s["V"], row_ptr, col, O=s["O"]), row_ptr, col
    idx = dsa.dsa_predict_mask(sh, s["Qt"], s["Kt"], idx=s["idx"], ws=s["ws"])
    S = dsa.dsa_sddmm(sh, s["Q"], s["K"], idx, S=s["S"])
    P = dsa.dsa_sparse_softmax(sh, S, P=s["P"])
    return dsa.dsa_spmm(sh, P, idx, s["V"], O=s["O"]), idx, S, P


def work(case):
    """Each input once, each output once; the scores of the selection (2 N L^2 k, per unit) and the products at the kept
    positions (4 N L keep d)."""
    c = case
    e = 4 if c["dtype"] == "f32" else 2
    rows = c["B"] * c["H"] * c["L"]
    units = rows // c["vec"]
    n = 3 * rows * c["d"] * e + 4 * rows * c["d"] + 4 * units * c["keep"]
    n += 2 * rows * c["k"] * c["bits"] // 8
    flops = 2 * units * c["L"] * c["k"] + 4 * rows * c["keep"] * c["d"]
    if c["op"] == "layer":
        n += 4 * c["d"] * c["k"]
        flops += 4 * rows * c["d"] * c["k"]
    if c["op"] == "threshold":
        n += 4 * units
    if c["op"] == "staged":
        n += 2 * 4 * rows * c["keep"]
    return {"bytes": n, "flops": flops}


def tolerance(case):
    """Masks and codes are whole numbers and exact.  Outputs: four times what the path differs from the same steps in
    64 bits over the listed cases and drawn ones (fp32: rel up to 3.3e-7 and largest 4.7e-6; bf16, where the softmax
    weights are rounded to bf16: 1.7e-3 and 0.013)."""
    return {"rel": 2e-6, "max": 2e-5} if case["dtype"] == "f32" else {"rel": 7e-3, "max": 0.05}
