"""Performance cases of the Sparse Linear Attention library: the calls a program makes through the package's public
entry points (`paper_2605_11354_amd.binding`), at the sizes of the benchmark configurations and of the ranges around them.

A case is a plain dict.  `kind` says what one pass is:
  forward    sla_forward
  train      sla_forward, then sla_wproj_grad (the gradient of the one trained parameter)
  reuse      sla_forward with its labels asked for, then the next layer on those labels (sla_forward_with_labels)
  alternate  a frame layer (B = frames) and a global layer (B = 1) on the same token-major activations, as the backbone
             alternates them
  qkv        sla_fp8_linear_qkv: the FP8 qkv projection that leaves Q, K and V in the attention's E4M3 form
  linear     sla_fp8_linear: the FP8 fake-quantised linear layer
  quantise   sla_quantise_e4m3 on Q, K and V
Inputs follow the benchmark's generator (tokens drawn from clusters that Q and K share, V ~ N(0,1)), drawn on the GPU.
"""
import math

import torch

from paper_2605_11354_amd import binding as B

DEV = "cuda:0"
FRAME = 1374          # tokens of a frame in the benchmark configurations: 1369 patches + 5 special tokens


def _attention(kind, Bn, H, N, bq, crit, neg, dtype="bf16", per_head=True, phi="softmax", layout="bhnd", clusters=256, **more):
    return dict(kind=kind, B=Bn, H=H, N=N, bq=bq, crit=crit, neg=neg, dtype=dtype, per_head=per_head, phi=phi, layout=layout,
                clusters=clusters, **more)


def listed():
    return [
        # smallest call: two heads, two small frames; launches and latency are all there is
        dict(_attention("forward", 1, 2, 512, 64, 0.125, 0.50, per_head=False, clusters=16), name="tiny"),
        # global attention over 8 frames, 64-row query blocks
        dict(_attention("forward", 1, 16, 8 * FRAME, 64, 0.05, 0.75), name="global8"),
        # global attention over 32 frames, the headline configuration
        dict(_attention("forward", 1, 16, 32 * FRAME, 128, 0.05, 0.80), name="global32"),
        # frame attention: every frame attends within itself
        dict(_attention("forward", 32, 16, FRAME, 64, 0.10, 0.60, clusters=64), name="frames32"),
        # E4M3 deployment path over 100 frames, the largest call
        dict(_attention("forward", 1, 16, 100 * FRAME, 128, 0.03, 0.85, dtype="fp8"), name="global100_e4m3"),
        # E4M3 frame attention on a few frames, token-major as the fused qkv projection leaves its heads
        dict(_attention("forward", 6, 16, FRAME, 64, 0.10, 0.60, dtype="fp8", layout="bnhd", clusters=64), name="frames6_e4m3"),
        # two layers sharing one set of block masks, a token count that fits no block, token-major
        dict(_attention("reuse", 1, 16, 13 * FRAME - 3, 128, 0.05, 0.80, per_head=False, layout="bnhd"), name="reuse13_ragged"),
        # training step of the projection: forward and gradient, with the feature map the algorithm prints
        dict(_attention("train", 1, 16, 8 * FRAME, 64, 0.05, 0.75, per_head=False, phi="elu1"), name="train8"),
        # one frame layer and one global layer of the backbone on the same activations
        dict(_attention("alternate", 8, 16, FRAME, 64, 0.10, 0.60, layout="bnhd", clusters=64, crit_global=0.05, neg_global=0.75),
             name="alternate8"),
        # qkv projection of the 32-frame layer into E4M3 Q, K, V
        dict(kind="qkv", B=1, N=32 * FRAME, H=16, d_in=1024, bq=128, bias=True, name="qkv32"),
        # qkv projection of a single frame as a plain layer
        dict(kind="linear", N=FRAME, d_in=1024, d_out=3072, bias=True, name="linear1"),
        # Q, K and V of the 32-frame layer to E4M3
        dict(kind="quantise", B=1, H=16, N=32 * FRAME, bq=128, layout="bhnd", name="quantise32"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["global", "global", "global_e4m3", "frames", "frames_e4m3", "train", "reuse", "alternate", "qkv", "linear",
                       "quantise"])
    H = rng.choice([2, 4, 8, 12, 16, 16])
    layout = rng.choice(["bhnd", "bnhd"])
    opts = dict(per_head=rng.random() < 0.5, phi=rng.choice(["softmax", "softmax", "softmax", "elu1"]), layout=layout)
    crit, neg = round(rng.uniform(0.03, 0.125), 3), round(rng.uniform(0.5, 0.85), 3)
    if kind in ("global", "global_e4m3", "train", "reuse"):
        fp8 = kind == "global_e4m3"
        top = {"global": 44000, "global_e4m3": 137400, "train": 44000, "reuse": 24000}[kind]
        # the share of critical blocks falls with the length, as in the configurations (12.5 % at 512 tokens to 3 % at 137400)
        N = _log_int(rng, 512, top)
        crit = min(crit, round(0.125 - 0.017 * math.log(N / 512), 3))
        name = kind if kind in ("train", "reuse") else "forward"
        return _attention(name, 1, H, N, rng.choice([64, 128]) if N < 20000 else 128, crit, neg, dtype="fp8" if fp8 else "bf16", **opts)
    if kind in ("frames", "frames_e4m3"):
        return _attention("forward", _log_int(rng, 2, 32), H, _log_int(rng, 300, 1800), 64, round(rng.uniform(0.05, 0.125), 3),
                          round(rng.uniform(0.5, 0.7), 3), dtype="fp8" if kind == "frames_e4m3" else "bf16", clusters=64, **opts)
    if kind == "alternate":
        opts["layout"] = "bnhd"
        return _attention("alternate", _log_int(rng, 2, 16), H, _log_int(rng, 300, 1500), 64, 0.10, 0.60, clusters=64,
                          crit_global=crit, neg_global=neg, **opts)
    if kind == "qkv":
        return dict(kind="qkv", B=1, N=_log_int(rng, 300, 44000), H=H, d_in=64 * max(H, 2), bq=rng.choice([64, 128]), bias=rng.random() < 0.7)
    if kind == "linear":
        return dict(kind="linear", N=_log_int(rng, 100, 44000), d_in=128 * rng.randint(2, 16), d_out=8 * _log_int(rng, 16, 512),
                    bias=rng.random() < 0.7)
    return dict(kind="quantise", B=rng.choice([1, 1, 4]), H=H, N=_log_int(rng, 500, 22000), bq=rng.choice([64, 128]), layout=layout)


# ------------------------------------------------------------------------------------------------------------ inputs
def _clustered(gen, Bn, H, N, clusters, own_centres):
    """Q, K, V [B,H,N,64] bf16: Q, K = 0.5 centre[cluster of the token] + N(0,1), V ~ N(0,1).  A token's cluster is the same
    in all heads; the batch items (frames) draw their own centres, or share them where a global layer joins the frames."""
    ids = torch.randint(0, clusters, (Bn, N), generator=gen, device=DEV)
    centres = torch.randn((Bn if own_centres else 1, H, clusters, 64), generator=gen, device=DEV).expand(Bn, H, clusters, 64)
    base = 0.5 * torch.gather(centres, 2, ids[:, None, :, None].expand(Bn, H, N, 64))
    q = (base + torch.randn((Bn, H, N, 64), generator=gen, device=DEV)).to(torch.bfloat16)
    k = (base + torch.randn((Bn, H, N, 64), generator=gen, device=DEV)).to(torch.bfloat16)
    v = torch.randn((Bn, H, N, 64), generator=gen, device=DEV).to(torch.bfloat16)
    return q, k, v


def _blocks(n, blk):
    return -(-n // blk)


def _quantised(x, blk, layout):
    Bn, H, N = (x.shape[0], x.shape[1], x.shape[2]) if layout == "bhnd" else (x.shape[0], x.shape[2], x.shape[1])
    codes = torch.empty(x.shape, dtype=torch.uint8, device=DEV)
    scales = torch.empty((Bn, H, _blocks(N, blk)), dtype=torch.float32, device=DEV)
    B.sla_quantise_e4m3(x, blk, codes, scales, layout=layout)
    return codes, scales


def _params(case, Bn=None, N=None, crit=None, neg=None):
    return B.make_params(Bn or case["B"], case["H"], N or case["N"], case["bq"], 64, crit or case["crit"], neg or case["neg"], -1, -1,
                         case["dtype"], case["per_head"], phi=case["phi"], layout=case["layout"])


def _tensors(case, gen):
    """(Q, K, V, sQ, sK, sV) in the case's layout and data type."""
    q, k, v = _clustered(gen, case["B"], case["H"], case["N"], case["clusters"], case["kind"] != "alternate")
    if case["layout"] == "bnhd":
        q, k, v = (t.transpose(1, 2).contiguous() for t in (q, k, v))
    if case["dtype"] == "bf16":
        return q, k, v, None, None, None
    (q, sq), (k, sk), (v, sv) = (_quantised(t, blk, case["layout"]) for t, blk in ((q, case["bq"]), (k, 64), (v, 64)))
    return q, k, v, sq, sk, sv


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    kind = case["kind"]
    st = {"kind": kind, "case": case}
    if kind in ("qkv", "linear"):
        N, d_in = case["N"], case["d_in"]
        d_out = 3 * case["H"] * 64 if kind == "qkv" else case["d_out"]
        st["x"] = torch.randn((N, d_in), generator=gen, device=DEV).to(torch.bfloat16)
        st["W"] = (torch.randn((d_out, d_in), generator=gen, device=DEV) / d_in ** 0.5).to(torch.bfloat16)
        st["bias"] = torch.randn((d_out,), generator=gen, device=DEV).to(torch.bfloat16) if case["bias"] else None
        # the layer's workspace: code matrices and scales of both operands (a program that serves keeps it)
        st["ws"] = torch.empty(N * (d_in + 4) + d_out * (d_in + 4) + 4096, dtype=torch.uint8, device=DEV)
        if kind == "linear":
            st["y"] = torch.empty((N, d_out), dtype=torch.bfloat16, device=DEV)
        else:
            H = case["H"]
            st["codes"] = [torch.empty((1, N, H, 64), dtype=torch.uint8, device=DEV) for _ in range(3)]
            st["scales"] = [torch.empty((1, H, _blocks(N, blk)), dtype=torch.float32, device=DEV) for blk in (case["bq"], 64, 64)]
        return st
    if kind == "quantise":
        shape = (case["B"], case["H"], case["N"], 64) if case["layout"] == "bhnd" else (case["B"], case["N"], case["H"], 64)
        st["x"] = [torch.randn(shape, generator=gen, device=DEV).to(torch.bfloat16) for _ in range(3)]
        st["codes"] = [torch.empty(shape, dtype=torch.uint8, device=DEV) for _ in range(3)]
        st["scales"] = [torch.empty((case["B"], case["H"], _blocks(case["N"], blk)), dtype=torch.float32, device=DEV) for blk in (case["bq"], 64, 64)]
        return st
    st["t"] = _tensors(case, gen)
    nW = case["H"] if case["per_head"] else 1
    W = (torch.randn((nW, 64, 64), generator=gen, device=DEV) / 8.0).to(torch.bfloat16)
    st["W"] = W if case["per_head"] else W[0].contiguous()
    st["p"] = _params(case)
    st["ws"] = B.alloc_workspace(st["p"])
    q = st["t"][0]
    st["O"] = torch.empty(q.shape, dtype=torch.bfloat16, device=DEV)
    if kind == "train":
        st["dO"] = torch.randn(q.shape, generator=gen, device=DEV).to(torch.bfloat16)
        st["dW"] = torch.empty((nW, 64, 64), dtype=torch.float32, device=DEV)
    elif kind == "reuse":
        # the second layer's Q and K are near the first one's, its V is its own; the masks of the first are used again
        q1, k1, v1 = st["t"][:3]
        near = lambda x: (x.float() + 0.25 * torch.randn(x.shape, generator=gen, device=DEV)).to(torch.bfloat16)
        st["t2"] = (near(q1), near(k1), torch.randn(v1.shape, generator=gen, device=DEV).to(torch.bfloat16), None, None, None)
        st["O2"] = torch.empty_like(st["O"])
        st["labels"] = torch.empty((case["B"], case["H"], _blocks(case["N"], case["bq"]), _blocks(case["N"], 64)), dtype=torch.int8, device=DEV)
    elif kind == "alternate":
        st["pg"] = _params(case, Bn=1, N=case["B"] * case["N"], crit=case["crit_global"], neg=case["neg_global"])
        st["ws"] = torch.empty(max(B.sla_workspace_bytes(st["p"]), B.sla_workspace_bytes(st["pg"])), dtype=torch.uint8, device=DEV)
        st["O2"] = torch.empty_like(st["O"])
    return st


# -------------------------------------------------------------------------------------------------------------- pass
def run(st):
    kind, case = st["kind"], st["case"]
    if kind == "linear":
        return {"y": B.sla_fp8_linear(st["x"], st["W"], st["bias"], st["y"], st["ws"])}
    if kind == "qkv":
        c, s = st["codes"], st["scales"]
        B.sla_fp8_linear_qkv(st["x"], st["W"], st["bias"], 1, case["N"], case["H"], case["bq"], c[0], c[1], c[2], s[0], s[1], s[2], st["ws"])
        return {"codes": c, "scales": s}
    if kind == "quantise":
        for x, blk, c, s in zip(st["x"], (case["bq"], 64, 64), st["codes"], st["scales"]):
            B.sla_quantise_e4m3(x, blk, c, s, layout=case["layout"])
        return {"codes": st["codes"], "scales": st["scales"]}
    q, k, v, sq, sk, sv = st["t"]
    if kind == "reuse":
        B.sla_forward(st["p"], q, k, v, st["W"], st["O"], st["labels"], sq, sk, sv, st["ws"])
        q2, k2, v2 = st["t2"][:3]
        B.sla_forward_with_labels(st["p"], q2, k2, v2, st["W"], st["labels"], st["O2"], None, None, None, st["ws"])
        return {"O": st["O"], "labels": st["labels"], "O2": st["O2"]}
    B.sla_forward(st["p"], q, k, v, st["W"], st["O"], None, sq, sk, sv, st["ws"])
    if kind == "train":
        B.sla_wproj_grad(st["p"], q, st["dO"], st["dW"], st["ws"], sq)
        return {"O": st["O"], "dW": st["dW"]}
    if kind == "alternate":
        B.sla_forward(st["pg"], q, k, v, st["W"], st["O2"], None, sq, sk, sv, st["ws"])
        return {"O": st["O"], "O2": st["O2"]}
    return {"O": st["O"]}


# -------------------------------------------------------------------------------------------------------------- work
def _forward_work(case, Bn, N, crit, neg, classify=True):
    BH, bq, es = Bn * case["H"], case["bq"], 1 if case["dtype"] == "fp8" else 2
    nq, nk = _blocks(N, bq), _blocks(N, 64)
    kc = min(nk, max(1, math.floor(crit * nk + 0.5)))
    km = nk - kc - min(nk - kc, math.floor(neg * nk + 0.5))
    nW = case["H"] if case["per_head"] else 1
    nbytes = BH * N * 64 * (3 * es + 2) + nW * 8192 + (BH * (nq + 2 * nk) * 4 if es == 1 else 0)
    flops = 4.0 * BH * N * min(N, kc * 64) * 64           # critical blocks
    flops += 2.0 * BH * N * 64 * 64 * 3                   # phi(K)^T V, phi(Q) H, projection
    flops += 1.0 * BH * nq * km * 65 * 64                 # sums of the marginal states
    if classify:
        flops += 2.0 * BH * nq * nk * 64
    return nbytes, flops


def work(case):
    kind = case["kind"]
    if kind in ("qkv", "linear"):
        N, d_in = case["N"], case["d_in"]
        d_out = 3 * case["H"] * 64 if kind == "qkv" else case["d_out"]
        out = N * d_out * 2 if kind == "linear" else N * d_out + case["H"] * (_blocks(N, case["bq"]) + 2 * _blocks(N, 64)) * 4
        return {"bytes": 2 * (N * d_in + d_out * d_in) + (2 * d_out if case["bias"] else 0) + out, "flops": 2.0 * N * d_in * d_out}
    if kind == "quantise":
        n = case["B"] * case["H"]
        return {"bytes": 9 * n * case["N"] * 64 + 4 * n * (_blocks(case["N"], case["bq"]) + 2 * _blocks(case["N"], 64)), "flops": 9.0 * n * case["N"] * 64}
    nbytes, flops = _forward_work(case, case["B"], case["N"], case["crit"], case["neg"])
    rows = case["B"] * case["H"] * case["N"]
    if kind == "train":
        nbytes += rows * 64 * 2 + (case["H"] if case["per_head"] else 1) * 16384          # dO in, dW out; Q was counted
        flops += 2.0 * rows * 64 * 64
    elif kind == "reuse":
        b2, f2 = _forward_work(case, case["B"], case["N"], case["crit"], case["neg"], classify=False)
        nbytes += b2 + case["B"] * case["H"] * _blocks(case["N"], case["bq"]) * _blocks(case["N"], 64)
        flops += f2
    elif kind == "alternate":
        b2, f2 = _forward_work(case, 1, case["B"] * case["N"], case["crit_global"], case["neg_global"])
        nbytes, flops = nbytes + rows * 64 * 2, flops + f2                                # the same Q, K, V; a second O
    return {"bytes": int(nbytes), "flops": float(flops)}


def tolerance(case):
    """About four times the error against the same arithmetic in fp64 (the oracle's, or the layer's exact products):
    O 1.7e-3 (2-norm) and 5.7e-3 (largest), nearly all of it the bf16 store; dW 2.1e-3 and 7.8e-3; y 1.7e-3 and 3.9e-3.  A y
    one bf16 unit off now and then (fp32 sums over d_in in another order) changes a code of the projection's output:
    1e-3 of them, and a block's scale where it is the largest entry (4e-4, 2-norm over the scales)."""
    kind = case["kind"]
    if kind == "quantise":
        return "exact"
    if kind == "qkv":
        return {"rel": 7e-3, "differ": 4e-3}
    if kind == "train":
        return {"rel": 8e-3, "max": 3e-2}
    if kind == "linear":
        return {"rel": 7e-3, "max": 1.6e-2}
    return {"rel": 7e-3, "max": 2.2e-2}
