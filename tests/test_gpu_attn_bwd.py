"""dQ, dK and dV of bf16 attention in tiles of 256 rows, where those tiles end: a block of one tile and a row more, last tiles with
one row, with one wave, with an odd half of a wave's 64 (D = 128: tiles of 128 keys, seeds in chunks of 256 rows), blocks of whole tiles, grouped query heads (their steps follow one another),
and enough heads that dQ takes these tiles too.  Against fp64 on the same bf16 rows (a head of each kind), at the parity suite's
bound for gradients."""
import math

import pytest
import torch

from paper_2509_10406_amd import binding as mb
from tests.util import bf16_grad_bound

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("N,Hq,Hkv", [(257, 1, 1), (320, 4, 1), (353, 3, 3), (512, 2, 1), (513, 4, 1), (545, 6, 3), (769, 8, 2), (1024, 48, 24), (1025, 32, 32), (1095, 33, 11),
                                      (1250, 30, 30), (1311, 28, 7)])
def test_tiles(N, Hq, Hkv, D):
    g = torch.Generator().manual_seed(N + D)
    p = mb.Params(B=1, Hq=Hq, Hkv=Hkv, N=N, D=D)
    Q, K, V, dO = (torch.randn(1, H, N, D, generator=g).bfloat16().cuda() for H in (Hq, Hkv, Hkv, Hq))
    O, LSE = mb.exact_attn_fwd(p, Q, K, V)
    got = mb.exact_attn_bwd(p, Q, K, V, O, LSE, dO)
    G = Hq // Hkv
    for hk in sorted({0, Hkv - 1}):
        k, v = K[0, hk].cpu().double(), V[0, hk].cpu().double()
        wk, wv = torch.zeros_like(k), torch.zeros_like(v)
        for h in range(hk * G, hk * G + G):
            q, d = Q[0, h].cpu().double(), dO[0, h].cpu().double()
            P = (q @ k.T / math.sqrt(D)).masked_fill(torch.ones(N, N, dtype=torch.bool).triu(1), -math.inf).softmax(-1)
            dP = d @ v.T
            dS = P * (dP - (P * dP).sum(-1, keepdim=True)) / math.sqrt(D)
            wq = dS @ k
            wk += dS.T @ q
            wv += P.T @ d
            assert (got[0][0, h].cpu().double() - wq).abs().max() <= bf16_grad_bound(float(wq.abs().max()))
        for x, w in ((got[1], wk), (got[2], wv)):
            assert (x[0, hk].cpu().double() - w).abs().max() <= bf16_grad_bound(float(w.abs().max()))


def test_a_row_that_is_not_finite_stays_with_its_successors():
    # a query row, and with it the keys it attends: its block's up to its own position, and no later ones
    g = torch.Generator().manual_seed(5)
    H, N, D = 32, 1100, 64
    p = mb.Params(B=1, Hq=H, Hkv=H, N=N, D=D)
    Q, K, V, dO = (torch.randn(1, H, N, D, generator=g).bfloat16().cuda() for _ in range(4))
    O, LSE = mb.exact_attn_fwd(p, Q, K, V)
    want = mb.exact_attn_bwd(p, Q, K, V, O, LSE, dO)
    n = 700
    dO[:, :, n, 3] = float("inf")
    dQ, dK, dV = mb.exact_attn_bwd(p, Q, K, V, O, LSE, dO)
    others = torch.arange(N, device="cuda") != n
    assert torch.equal(dQ[:, :, others], want[0][:, :, others])
    far = torch.arange(N, device="cuda") >= (n // 64 + 1) * 64  # the matrix instructions meet a masked pair inside 64 rows
    assert torch.equal(dK[:, :, far], want[1][:, :, far]) and torch.equal(dV[:, :, far], want[2][:, :, far])


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("odd", ["Q", "K", "V", "dO"])
def test_tensors_off_a_16_byte_boundary(odd, D):
    # a view one element into its storage: the kernels of 128 rows, with gradients in either type.  dK and dV add up in the same
    # order there; dQ takes its key tiles the other way round: the same products, N of them, added in fp32 (2^-24 each of what has
    # been added up, which stays below 16 times the largest entry for rows like these).
    g = torch.Generator().manual_seed(D)
    H, N = 32, 1100
    t = {n: torch.randn(1, H, N, D, generator=g).bfloat16().cuda() for n in ("Q", "K", "V", "dO")}
    args = lambda: (t["Q"], t["K"], t["V"], O, LSE, t["dO"])
    p = mb.Params(B=1, Hq=H, Hkv=H, N=N, D=D)
    p16 = mb.Params(B=1, Hq=H, Hkv=H, N=N, D=D, grad_dtype=mb.BF16)
    O, LSE = mb.exact_attn_fwd(p, t["Q"], t["K"], t["V"])
    want = mb.exact_attn_bwd(p, *args())
    x = torch.empty(t[odd].numel() + 8, dtype=torch.bfloat16, device="cuda")[1:1 + t[odd].numel()].view(t[odd].shape)
    t[odd] = x.copy_(t[odd])
    got = mb.exact_attn_bwd(p, *args())
    assert torch.equal(got[1], want[1]) and torch.equal(got[2], want[2])
    assert (got[0] - want[0]).abs().max() <= 16 * N * 2.0 ** -24 * want[0].abs().max()
    assert all(torch.equal(a, b.bfloat16()) for a, b in zip(mb.exact_attn_bwd(p16, *args()), got))
