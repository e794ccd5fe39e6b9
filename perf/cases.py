"""What the framework's speed is measured on: calls that a user's program makes through the public entry points
(`paper_2509_10406_amd.binding`), over the range of sizes, types and options that the repository's own workloads,
tests and benchmark cover.

A case is a dict of plain values.  Its `path` says which calls one pass makes:
  "train"  muse_cluster + muse_fwd + muse_bwd: a layer of a training step, the forward's state kept for the backward
  "eval"   muse_cluster + muse_fwd: a layer of an evaluation pass
  "exact"  exact_attn_fwd + exact_attn_bwd: the exact attention that the method is compared with
The other values are the fields of `Params`, plus `gen`, the kind of activations the inputs imitate (see `prepare`).
"""
import math

import torch

from paper_2509_10406_amd import binding as mb


def _case(name, path, gen, **kw):
    c = dict(name=name, path=path, gen=gen, B=1, Hq=1, Hkv=1, N=2048, D=64, Cq=1, Ck=1, r=0, k2=1, block=0, iters=10,
             dtype="bf16", grad="fp32", streaming=False, balanced=False)
    c.update(kw)
    return c


def listed():
    return [
        # one head in fp32 at 2k tokens: the smallest call, as in a unit test or a first look at the method
        _case("eval_2k_fp32", "eval", "mixture", N=2048, Cq=16, Ck=32, r=2, dtype="fp32"),
        # fp32 training at a size where one still debugs or checks gradients
        _case("train_8k_fp32", "train", "mixture", Hq=4, Hkv=4, N=8192, Cq=32, Ck=128, r=4, dtype="fp32"),
        # odd sizes throughout (block 749, cluster counts that fill no tile), two sequences, two retrieved blocks,
        # gradients in bf16: a variable-length fine-tuning batch
        _case("train_6k_ragged", "train", "embed", B=2, Hq=6, Hkv=3, N=5992, Cq=23, Ck=71, r=5, k2=2, grad="bf16"),
        # a small model's layer
        _case("train_16k", "train", "embed", Hq=8, Hkv=8, N=16384, Cq=64, Ck=256, r=4),
        # the 1B-scale pretraining layer that the benchmark times
        _case("train_64k", "train", "embed", Hq=16, Hkv=16, N=65536, Cq=256, Ck=1024, r=8),
        # the same layer at the paper's operating ratio, clusters = N / 512
        _case("train_64k_qk128", "train", "embed", Hq=16, Hkv=16, N=65536, Cq=128, Ck=128, r=8),
        # grouped queries with rotary keys: the largest call
        _case("train_64k_gqa", "train", "rope", Hq=32, Hkv=8, N=65536, Cq=256, Ck=1024, r=8),
        # head dimension 128 with grouped queries, clusters and retrieval in the proportions of a 128k layer
        _case("train_32k_d128", "train", "rope", Hq=32, Hkv=8, N=32768, D=128, Cq=128, Ck=512, r=16),
        # the paper's own clustering: one streaming pass and the cap on clusters per block
        _case("train_32k_streaming", "train", "embed", Hq=16, Hkv=16, N=32768, Cq=64, Ck=64, r=4, streaming=True,
              balanced=True),
        # evaluation of a head-dimension-128 layer at the operating ratio
        _case("eval_32k_d128", "eval", "rope", Hq=32, Hkv=8, N=32768, D=128, Cq=64, Ck=64, r=4),
        # exact attention, forward and backward, at the small model's layer ...
        _case("exact_16k", "exact", "embed", Hq=8, Hkv=8, N=16384),
        # ... and with head dimension 128, grouped queries and gradients in bf16
        _case("exact_8k_d128", "exact", "rope", Hq=32, Hkv=8, N=8192, D=128, grad="bf16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the ranges above: any path, 1k to 64k tokens (fp32: to 8k), 1 to 32 heads, both head dimensions."""
    largest = work(_case("", "train", "rope", Hq=32, Hkv=8, N=65536, Cq=256, Ck=1024, r=8))["flops"]
    while True:
        path = rng.choice(["train", "train", "train", "eval", "exact"])
        dtype = rng.choice(["bf16", "bf16", "bf16", "fp32"])
        D = rng.choice([64, 64, 128])
        group = rng.choice([1, 1, 2, 4])
        if dtype == "fp32":
            Hkv, block, nb = rng.randint(1, 4), _log_int(rng, 128, 1024), 8
            group = min(group, 2)
        else:
            Hkv, block, nb = _log_int(rng, 1, 16), _log_int(rng, 128, 8192), rng.choice([8, 8, 8, 4, 12])
        N = block * nb
        c = _case("", path, rng.choice(["embed", "rope"]) if dtype == "bf16" else "mixture", B=rng.choice([1, 1, 2]),
                  Hq=Hkv * group, Hkv=Hkv, N=N, D=D, dtype=dtype,
                  grad=rng.choice(["fp32", "bf16"]) if dtype == "bf16" else "fp32")
        del c["name"]
        if path != "exact":
            c["block"] = block
            c["Cq"] = max(2, min(256, int(N / rng.uniform(200, 560))))
            c["Ck"] = max(4, min(1024, int(c["Cq"] * rng.choice([1, 1, 2, 3, 4]) * rng.uniform(0.8, 1.2))))
            c["r"] = rng.choice([0, 1, 2, 4, 4, 5, 8, 8, 16])
            c["k2"] = rng.choice([1, 1, 1, 2])
            c["iters"] = rng.choice([1, 5, 10])
            c["streaming"] = dtype == "bf16" and N <= 32768 and rng.random() < 0.1
            c["balanced"] = 4 * block // max(c["Cq"], c["Ck"]) >= 2 and rng.random() < 0.1
            if c["r"] > c["Ck"]:
                continue
        # no larger than the largest listed one, in work (fp32 runs at a small part of the bf16 rate) and in memory
        if work(c)["flops"] * (16 if dtype == "fp32" else 1) > largest:
            continue
        if N > 65536 or c["B"] * c["Hq"] * (nb - 1) * c["Cq"] * c["Ck"] * D > 32 * 7 * 256 * 1024 * 64:
            continue
        return c


def _params(c):
    flags = mb.FLAG_KEEP_FWD_STATE if c["path"] == "train" else 0
    flags |= (mb.FLAG_STREAMING_KMEANS if c["streaming"] else 0) | (mb.FLAG_BALANCED_ASSIGN if c["balanced"] else 0)
    return mb.Params(B=c["B"], Hq=c["Hq"], Hkv=c["Hkv"], N=c["N"], D=c["D"], Cq=c["Cq"], Ck=c["Ck"], r=c["r"], k2=c["k2"],
                     block=c["block"], kmeans_iters=c["iters"], dtype=mb.BF16 if c["dtype"] == "bf16" else mb.FP32,
                     grad_dtype=mb.BF16 if c["grad"] == "bf16" else mb.FP32, flags=flags)


def _mixture(g, n, dim, components, sd=0.3):
    dev = g.device
    centres = torch.randn(components, dim, generator=g, device=dev)
    comp = torch.randint(0, components, (n,), generator=g, device=dev)
    return centres[comp] + sd * torch.randn(n, dim, generator=g, device=dev)


def _rotary(x, base=1.0e5):
    """Rotary phase at position n on the pairs (2t, 2t+1), theta_t = base^(-2t/D).  x: [B, H, N, D]."""
    N, D = x.shape[-2:]
    t = torch.arange(D // 2, dtype=torch.float64, device=x.device)
    ang = torch.arange(N, dtype=torch.float64, device=x.device)[:, None] * base ** (-2.0 * t / D)
    cs, sn = torch.cos(ang).float(), torch.sin(ang).float()
    xe, xo = x[..., 0::2], x[..., 1::2]
    return torch.stack((xe * cs - xo * sn, xe * sn + xo * cs), dim=-1).flatten(-2)


def prepare(case, seed):
    """The layer's activations and the seeded shuffle that the clustering starts from (every floor(N/C)-th position).
    The activations are one of three kinds:
      mixture  every head's rows from a Gaussian mixture of its own (the clusters are there to be found)
      embed    projections of token embeddings, the tokens being drawn from a mixture: as in a layer, the heads and
               Q, K, V of one position share the token
      rope     the same with rotary phases on Q and K: position turns the row, clusters are harder to find"""
    c, p = case, _params(case)
    B, N, D = c["B"], c["N"], c["D"]
    g = torch.Generator(device="cuda").manual_seed(seed)
    heads = (c["Hq"], c["Hkv"], c["Hkv"])
    if c["gen"] == "mixture":
        rows = [torch.stack([_mixture(g, N, D, 16) for _ in range(B * H)]).view(B, H, N, D) for H in heads]
    else:
        E = 512
        emb = torch.stack([_mixture(g, N, E, max(16, min(1024, N // 64))) for _ in range(B)])
        rows = [(emb @ (torch.randn(E, H * D, generator=g, device="cuda") / math.sqrt(E))).view(B, N, H, D).transpose(1, 2)
                for H in heads]
        if c["gen"] == "rope":
            rows[:2] = [_rotary(x) for x in rows[:2]]
    s = {"path": c["path"], "p": p}
    for name, x in zip("QKV", rows):
        s[name] = x.to(p.torch_dtype).contiguous()
    if c["path"] != "eval":
        s["dO"] = torch.randn(B, c["Hq"], N, D, generator=g, device="cuda").to(p.torch_dtype)
    if c["path"] != "exact":
        for name, H, C in (("qi", c["Hq"], c["Cq"]), ("ki", c["Hkv"], c["Ck"])):
            at = torch.rand(B, H, N, generator=g, device="cuda").argsort(-1)
            s[name] = at[..., torch.arange(C, device="cuda") * (N // C)].to(torch.int32).contiguous()
    return s


def run(state):
    s, p = state, state["p"]
    if s["path"] == "exact":
        O, LSE = mb.exact_attn_fwd(p, s["Q"], s["K"], s["V"])
        dQ, dK, dV = mb.exact_attn_bwd(p, s["Q"], s["K"], s["V"], O, LSE, s["dO"])
        return {"O": O, "LSE": LSE, "dQ": dQ, "dK": dK, "dV": dV}
    qc, qa, kc, ka = mb.muse_cluster(p, s["Q"], s["K"], s["qi"], s["ki"])
    O, LSE, selc, selb = mb.muse_fwd(p, s["Q"], s["K"], s["V"], qc, qa, ka)
    out = {"qc": qc, "qa": qa, "kc": kc, "ka": ka, "O": O, "LSE": LSE}
    if p.r:
        out["selc"], out["selb"] = selc, selb
    if s["path"] == "train":
        out["dQ"], out["dK"], out["dV"] = mb.muse_bwd(p, s["Q"], s["K"], s["V"], O, LSE, s["dO"], qc, qa, ka, selc, selb)
    return out


def work(case):
    """Inputs read once, outputs written once; the products of the method: nearest centroids in every pass over the
    rows, N x C x D products of the monopole (5 forward, 12 backward), the retrieved pairs, and attention inside a block
    (2 products forward, 5 backward, half of each behind the causal mask).  For "exact" the block is the sequence."""
    c = case
    B, Hq, Hkv, N, D = c["B"], c["Hq"], c["Hkv"], c["N"], c["D"]
    es, gs = (2 if c["dtype"] == "bf16" else 4), (2 if c["grad"] == "bf16" else 4)
    bwd = c["path"] != "eval"
    q, k = B * Hq * N * D, B * Hkv * N * D
    byts = (q + 2 * k) * es + q * es + B * Hq * N * 4
    if bwd:
        byts += q * es + (q + 2 * k) * gs
    block = N if c["path"] == "exact" else c["block"] or N // 8
    flops = (7 if bwd else 2) * q * block
    if c["path"] != "exact":
        nb = N // block
        far = (nb - 1) / nb
        passes = 2 if c["streaming"] else c["iters"] + 1
        flops += 2 * passes * (q * c["Cq"] + k * c["Ck"])
        flops += (17 if bwd else 5) * q * far * (3 * c["Cq"] + 2 * c["Ck"]) / 5 * 2
        flops += (14 if bwd else 4) * q * far * c["r"] * c["k2"] * block / c["Ck"]
        byts += 4 * (B * Hq * N * (1 + c["r"] + c["r"] * c["k2"]) + B * Hkv * N + D * (B * Hq * c["Cq"] + B * Hkv * c["Ck"]))
    return {"bytes": byts, "flops": flops}


def tolerance(case):
    """Measured by running the path on rows whose head dimensions are permuted (the same mathematics, every dot product
    summed in another order) and, for bf16, against the fp32 path on the same rows.
      exact  bf16: 2.8e-3 of the norm, 0.12 of the root mean square at most; fp32: 6e-7
      with clustering: Lloyd iterations amplify a last-bit difference in a centroid (another row of its cluster, another
      cluster retrieved for a query), 1e-4 to 4e-2 of the norm and a whole value in single rows; with the same
      partition 3e-4 of the norm, 0.7 in single rows, and 1e-5 of the retrieved clusters differ (ties)"""
    if case["path"] == "exact":
        return {"rel": 1e-2, "max": 0.5} if case["dtype"] == "bf16" else {"rel": 1e-5, "max": 1e-4}
    return {"rel": 0.03, "max": 0.99, "differ": 0.01}
