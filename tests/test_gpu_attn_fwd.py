"""bf16 attention forward where its schedule changes: fewer rows than a tile, partial key steps, blocks that do not line up
with tiles, workgroups that take a tile and its mirror (an odd number of tiles leaves one without), and scores that make the
softmax reference move in every step, in none, or by more than fp32's range.  Against fp64 on the same bf16 rows: |O| is at
most max |v|, its error at most the rounding of P and O to bf16 (2 x 2^-9 of the largest value of a row's keys) plus the fp32
scores' share; 2e-2 as in the rest of the suite (values here stay below 4)."""
import pytest
import torch

from paper_2509_10406_amd import binding as mb

pytestmark = pytest.mark.gpu


def check(Q, K, V, scale=0.0):
    B, H, N, D = Q.shape
    p = mb.Params(B=B, Hq=H, Hkv=K.shape[1], N=N, D=D, scale=scale)
    O, LSE = mb.exact_attn_fwd(p, Q, K, V)
    g = H // K.shape[1]
    mask = torch.ones(N, N, dtype=torch.bool, device="cuda").triu(1)
    for h in range(H):
        q, k, v = (x[0, i].double() for x, i in ((Q, h), (K, h // g), (V, h // g)))
        s = (q @ k.T * (scale or D ** -0.5)).masked_fill(mask, float("-inf"))
        lse = torch.logsumexp(s, -1)
        o = torch.exp(s - lse[:, None]) @ v
        assert (O[0, h].double() - o).abs().max() <= 2e-2
        assert ((LSE[0, h].double() - lse).abs() <= 2e-2 + 1e-5 * lse.abs()).all()


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("N,H,Hkv", [(1, 1, 1), (33, 2, 1), (64, 1, 1), (257, 2, 2), (700, 3, 1), (1030, 88, 11), (512, 256, 32)])
def test_sizes(N, H, Hkv, D):
    g = torch.Generator(device="cuda").manual_seed(N + D)
    r = lambda h: torch.randn(1, h, N, D, generator=g, device="cuda").clamp(-4, 4).to(torch.bfloat16)
    check(r(H), r(Hkv), r(Hkv))


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("kind", ["rising", "falling", "huge", "tiny"])
def test_reference_moves(kind, D):
    N = 600
    g = torch.Generator(device="cuda").manual_seed(D)
    r = lambda: torch.randn(1, 1, N, D, generator=g, device="cuda").clamp(-4, 4)
    Q, K, V = r(), r(), r()
    n = torch.arange(N, device="cuda")[:, None]
    if kind in ("rising", "falling"):  # along the keys every score moves by about 30 per step of 64
        Q[..., 0], K[..., :1] = 8.0, (n if kind == "rising" else N - n) * (0.5 * D ** 0.5 / 8)
    elif kind == "huge":  # scores of 1e4: one key takes all
        Q, K = 40 * Q, 40 * K
    else:  # all scores far below zero: p = exp(s) alone would vanish
        Q[..., 0], K[..., 0] = 100.0, -20.0
    check(Q.to(torch.bfloat16), K.to(torch.bfloat16), V.to(torch.bfloat16))
