"""dQ of bf16 attention where its staging changes: one step of 64 keys, a step more or a key more than that, the last step
partly past the end, waves that end before the workgroup does, grouped queries.  Against fp64 on the same bf16 rows, at the
parity suite's bound for gradients."""
import math

import pytest
import torch

from paper_2509_10406_amd import binding as mb
from tests.util import bf16_grad_bound

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("N,Hq,Hkv", [(1, 1, 1), (63, 1, 1), (64, 2, 1), (65, 1, 1), (128, 2, 2), (193, 4, 2), (450, 9, 3)])
def test_steps(N, Hq, Hkv, D):
    g = torch.Generator().manual_seed(N + D)
    p = mb.Params(B=1, Hq=Hq, Hkv=Hkv, N=N, D=D)
    Q, K, V, dO = (torch.randn(1, H, N, D, generator=g).bfloat16().cuda() for H in (Hq, Hkv, Hkv, Hq))
    O, LSE = mb.exact_attn_fwd(p, Q, K, V)
    dQ = mb.exact_attn_bwd(p, Q, K, V, O, LSE, dO)[0]
    q, k, v, d = (x.cpu().double() for x in (Q, K, V, dO))
    k, v = k.repeat_interleave(Hq // Hkv, 1), v.repeat_interleave(Hq // Hkv, 1)
    S = (q @ k.transpose(-1, -2)) / math.sqrt(D)
    P = S.masked_fill(torch.ones(N, N, dtype=torch.bool).triu(1), -math.inf).softmax(-1)
    dP = d @ v.transpose(-1, -2)
    want = P * (dP - (P * dP).sum(-1, keepdim=True)) @ k / math.sqrt(D)
    assert (dQ.cpu().double() - want).abs().max() <= bf16_grad_bound(float(want.abs().max()))
