"""Exact attention of fp32 inputs at the edges of its tiles (16 rows or columns per wave, 64 per workgroup, 64 or 32 staged
rows), grouped queries and both head dims, against float64.  Tolerance: the parity suite's 1e-4 of the largest entry."""
import math

import pytest
import torch

from paper_2509_10406_amd import binding as mb
from tests.util import FP32_REL

pytestmark = pytest.mark.gpu


def reference(p, Q, K, V, dO):
    G = p.Hq // p.Hkv
    Q, K, V = (x.cpu().double().requires_grad_() for x in (Q, K, V))
    k, v = K.repeat_interleave(G, 1), V.repeat_interleave(G, 1)
    S = (Q @ k.transpose(-1, -2)) / math.sqrt(p.D)
    S = S.masked_fill(torch.ones(p.N, p.N, dtype=torch.bool).triu(1), -math.inf)
    O = S.softmax(-1) @ v
    O.backward(dO.cpu().double())
    return O.detach(), S.logsumexp(-1).detach(), Q.grad, K.grad, V.grad


def inputs(N, D, Hq, Hkv):
    g = torch.Generator().manual_seed(N + D)
    p = mb.Params(B=1, Hq=Hq, Hkv=Hkv, N=N, D=D, Cq=1, Ck=1, r=0, k2=1, block=0, kmeans_iters=0, dtype=mb.FP32, grad_dtype=mb.FP32)
    return p, [torch.randn(1, H, N, D, generator=g).cuda() for H in (Hq, Hkv, Hkv, Hq)]


@pytest.mark.parametrize("N,D,Hq,Hkv", [(1, 64, 1, 1), (15, 64, 2, 1), (17, 128, 1, 1), (64, 64, 1, 1), (65, 128, 2, 2),
                                        (127, 64, 3, 1), (300, 128, 4, 2), (1029, 64, 17, 17)])
def test_exact_fp32(N, D, Hq, Hkv):
    p, (Q, K, V, dO) = inputs(N, D, Hq, Hkv)
    O, LSE = mb.exact_attn_fwd(p, Q, K, V)
    got = (O, LSE, *mb.exact_attn_bwd(p, Q, K, V, O, LSE, dO))
    for name, a, b in zip(("O", "LSE", "dQ", "dK", "dV"), got, reference(p, Q, K, V, dO)):
        # a single row has dQ = dK = 0: what remains is p (dO . v - delta) k / sqrt(D), the difference of two sums of D = 64
        # products rounded at 2^-24 each, below 64 * 2^-24 * sum|dO v| (about 40) * |k| / 8 (about 0.4) = 6e-5 of unit rows
        err = (a.cpu().double() - b).abs().max() / b.abs().max().clamp(min=1.0)
        assert err <= FP32_REL, (name, float(err))


def test_later_infinities_stay_out():
    """A value row that is not finite reaches the queries from its position on, and no earlier one."""
    p, (Q, K, V, dO) = inputs(200, 64, 1, 1)
    O0, _ = mb.exact_attn_fwd(p, Q, K, V)
    V[0, 0, 70] = math.inf
    O, LSE = mb.exact_attn_fwd(p, Q, K, V)
    assert torch.allclose(O[:, :, :70], O0[:, :, :70], rtol=1e-6, atol=1e-6) and not O[:, :, 70:].isfinite().any()
    dQ, dK, dV = mb.exact_attn_bwd(p, Q, K, V, O0, LSE, dO)
    assert dQ[:, :, :70].isfinite().all()


def test_attended_infinity_with_a_vanishing_weight():
    """A query whose weight of a value row that is not finite underflows to zero still attends it: 0 * inf, on every tile."""
    p, (Q, K, V, _) = inputs(40, 64, 1, 1)
    Q[..., 0], K[..., 0] = 40.0, 1.0
    K[0, 0, 5, 0], V[0, 0, 5] = -40.0, math.inf      # a score of -200 against some 5
    O, _ = mb.exact_attn_fwd(p, Q, K, V)
    assert O[:, :, :5].isfinite().all() and not O[:, :, 5:].isfinite().any()


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("what", ["dO", "Q"])
def test_earlier_infinities_stay_out_of_later_keys(what, D):
    """A query row that is not finite reaches dK and dV of the keys up to its position; those of the later keys are what they
    are without that row."""
    p, (Q, K, V, dO) = inputs(200, D, 4, 2)
    O, LSE = mb.exact_attn_fwd(p, Q, K, V)
    for n in (0, 37, 130):                            # in the second query head of the first group
        without, Qi, gi = dO.clone(), Q.clone(), dO.clone()
        without[0, 1, n] = 0.0
        (gi if what == "dO" else Qi)[0, 1, n] = math.inf
        _, dK0, dV0 = mb.exact_attn_bwd(p, Q, K, V, O, LSE, without)
        _, dK, dV = mb.exact_attn_bwd(p, Qi, K, V, O, LSE, gi)
        assert dK.isfinite()[:, 1].all() and dK.isfinite()[:, :, n + 1:].all() and dV.isfinite()[:, :, n + 1:].all()
        for a, b in ((dK, dK0), (dV, dV0)):
            err = (a - b).abs()[:, :, n + 1:].max() / b.abs().max()
            assert err <= FP32_REL, float(err)
        assert not dK[:, 0, : n + 1].isfinite().all()
