"""The small kernels around bf16 and fp32 attention: row sums dO . O and the casts of the gradients, where their wide forms give
way to the narrow ones (an O or a result that does not start at a 16-byte boundary: the same values) and where their last
workgroup has rows left over.  The row sums are checked through dQ of one block, against fp64."""
import math

import pytest
import torch

from paper_2509_10406_amd import binding as mb
from tests.util import bf16_grad_bound

pytestmark = pytest.mark.gpu


def _offset(x):
    """The same values one element behind a 16-byte boundary."""
    y = torch.empty(x.numel() + 8, dtype=x.dtype, device=x.device)[1:1 + x.numel()].view(x.shape)
    y.copy_(x)
    return y


@pytest.mark.parametrize("D", [64, 128])
def test_bf16_gradients_of_long_blocks(D):
    # written by the attention kernels themselves (odd results: cast from fp32): the fp32 gradients, rounded once
    g = torch.Generator().manual_seed(D)
    H, Hkv, N = 34, 17, 1100
    Q, K, V, dO = (torch.randn(1, h, N, D, generator=g).bfloat16().cuda() for h in (H, Hkv, Hkv, H))
    p = mb.Params(B=1, Hq=H, Hkv=Hkv, N=N, D=D)
    p16 = mb.Params(B=1, Hq=H, Hkv=Hkv, N=N, D=D, grad_dtype=mb.BF16)
    O, LSE = mb.exact_attn_fwd(p, Q, K, V)
    want = tuple(x.bfloat16() for x in mb.exact_attn_bwd(p, Q, K, V, O, LSE, dO))
    assert all(torch.equal(a, b) for a, b in zip(mb.exact_attn_bwd(p16, Q, K, V, O, LSE, dO), want))
    out = tuple(_offset(torch.zeros_like(x)) for x in want)
    mb.exact_attn_bwd(p16, Q, K, V, O, LSE, dO, out=out)
    assert all(torch.equal(a, b) for a, b in zip(out, want))


@pytest.mark.parametrize("dtype", [mb.BF16, mb.FP32])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("N,H", [(1, 1), (33, 3), (127, 1), (130, 5)])
def test_row_sums_and_casts(N, H, D, dtype):
    g = torch.Generator().manual_seed(N + D)
    p = mb.Params(B=1, Hq=H, Hkv=H, N=N, D=D, dtype=dtype, grad_dtype=dtype)
    Q, K, V, dO = (torch.randn(1, H, N, D, generator=g).to(p.torch_dtype).cuda() for _ in range(4))
    O, LSE = mb.exact_attn_fwd(p, Q, K, V)
    got = mb.exact_attn_bwd(p, Q, K, V, O, LSE, dO)
    again = mb.exact_attn_bwd(p, Q, K, V, _offset(O), LSE, dO)
    assert all(torch.equal(a, b) for a, b in zip(got, again))
    if dtype == mb.BF16:
        out = tuple(_offset(torch.zeros_like(x)) for x in got)
        mb.exact_attn_bwd(p, Q, K, V, O, LSE, dO, out=out)
        assert all(torch.equal(a, b) for a, b in zip(got, out))
    q, k, v, d = (x[0].cpu().double() for x in (Q, K, V, dO))
    P = (q @ k.transpose(1, 2) / math.sqrt(D)).masked_fill(torch.ones(N, N, dtype=torch.bool).triu(1), -math.inf).softmax(-1)
    dP = d @ v.transpose(1, 2)
    want = (P * (dP - (P * dP).sum(-1, keepdim=True))) @ k / math.sqrt(D)
    bound = bf16_grad_bound(float(want.abs().max())) if dtype == mb.BF16 else 1e-5 * max(1.0, float(want.abs().max()))
    assert (got[0][0].cpu().double() - want).abs().max() <= bound


@pytest.mark.parametrize("odd,launches", [((), 1), ((2,), 2), ((0, 1), 3), ((0, 1, 2), 3)])
def test_one_gradient_off_the_boundary(odd, launches):
    # it goes through the narrow kernel alone: the others keep the wide one, in one launch
    g = torch.Generator().manual_seed(7)
    p = mb.Params(B=1, Hq=2, Hkv=2, N=130, D=64, grad_dtype=mb.BF16)
    Q, K, V, dO = (torch.randn(1, 2, 130, 64, generator=g).bfloat16().cuda() for _ in range(4))
    O, LSE = mb.exact_attn_fwd(p, Q, K, V)
    want = mb.exact_attn_bwd(p, Q, K, V, O, LSE, dO)
    out = tuple(_offset(torch.zeros_like(x)) if i in odd else torch.zeros_like(x) for i, x in enumerate(want))
    mb.muse_profile_enable(True)
    try:
        mb.exact_attn_bwd(p, Q, K, V, O, LSE, dO, out=out)
        assert mb.muse_profile_report()["k_cast"][0] == launches
    finally:
        mb.muse_profile_enable(False)
    assert all(torch.equal(a, b) for a, b in zip(out, want))


@pytest.mark.parametrize("D,N", [(64, 1100), (128, 1100), (64, 300)])
@pytest.mark.parametrize("on", [("dO", None, None), (None, "K", "V"), ("Q", "K", "V"), ("O", "V", "K"), ("dO half", None, None)])
def test_bf16_gradients_on_the_inputs(on, D, N):
    # gradients that replace the tensors they are made from: the values of gradients in memory of their own, also in the long
    # blocks whose kernels write bf16 gradients one after the other
    g = torch.Generator().manual_seed(D)
    H = 34
    t = {n: torch.randn(1, H, N, D, generator=g).bfloat16().cuda() for n in ("Q", "K", "V", "dO")}
    p = mb.Params(B=1, Hq=H, Hkv=H, N=N, D=D, grad_dtype=mb.BF16)
    t["O"], LSE = mb.exact_attn_fwd(p, t["Q"], t["K"], t["V"])
    want = mb.exact_attn_bwd(p, t["Q"], t["K"], t["V"], t["O"], LSE, t["dO"])
    if on[0] == "dO half":  # dQ begins in the middle of dO
        both = torch.empty(t["dO"].numel() * 3 // 2, dtype=torch.bfloat16, device="cuda")
        n = t["dO"].numel()
        both[:n] = t["dO"].flatten()
        t["dO"], t["dO half"] = both[:n].view(1, H, N, D), both[n // 2:].view(1, H, N, D)
    out = tuple(torch.empty_like(w) if x is None else t[x] for x, w in zip(on, want))
    mb.exact_attn_bwd(p, t["Q"], t["K"], t["V"], t["O"], LSE, t["dO"], out=out)
    assert all(torch.equal(a, b) for a, b in zip(out, want))
