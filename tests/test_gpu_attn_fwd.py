"""bf16 attention forward where its schedule changes: fewer rows than a tile, partial key steps, blocks that are no multiple of
the tile of 256 rows (waves without a query, partial last tiles, blocks smaller than a wave's 32 queries), workgroups that take
a tile and its mirror or are numbered across groups, and scores that make the softmax reference move in every step,
in none, or by more than fp32's range.  Against fp64 on the same bf16 rows: |O| is at
most max |v|, its error at most the rounding of P and O to bf16 (2 x 2^-9 of the largest value of a row's keys) plus the fp32
scores' share; 2e-2 as in the rest of the suite (values here stay below 4)."""
import pytest
import torch

import tests.test_gpu_muse as base
from paper_2509_10406_amd import binding as mb
from paper_2509_10406_amd.inputs import generate, small

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


def test_more_heads_than_a_grid_dimension_has_rows():
    g = torch.Generator(device="cuda").manual_seed(1)
    B = 66000  # 528000 heads, eight to a row of the grid
    Q, K, V = (torch.randn(B, 8, 1, 64, generator=g, device="cuda").bfloat16() for _ in range(3))
    O = mb.exact_attn_fwd(mb.Params(B=B, Hq=8, Hkv=8, N=1, D=64), Q, K, V)[0]
    assert torch.equal(O, V)  # one key: its weight is 1


BLOCKS = {
    "fwd_block384_d128": ("cfg2", dict(D=128, N=1152, Hq=2, Hkv=1, Cq=6, Ck=20, r=3, block=384, kmeans_iters=1)),
    "fwd_block128_d128": ("cfg2", dict(D=128, N=640, Hq=1, Hkv=1, Cq=4, Ck=12, r=2, block=128, kmeans_iters=1)),
    "fwd_block300": ("cfg2", dict(N=900, Hq=2, Hkv=2, Cq=5, Ck=17, r=2, block=300, kmeans_iters=1)),
    "fwd_block700": ("cfg2", dict(N=1400, Hq=2, Hkv=1, Cq=7, Ck=33, r=4, block=700, kmeans_iters=1)),
    "fwd_block20": ("cfg2", dict(N=320, Hq=1, Hkv=1, Cq=2, Ck=6, r=1, block=20, kmeans_iters=1)),
    "fwd_block1": ("cfg2", dict(D=128, N=16, Hq=1, Hkv=1, Cq=1, Ck=2, r=1, block=1, kmeans_iters=1)),
}


@pytest.mark.parametrize("name", list(BLOCKS))
def test_blocks(name, monkeypatch):
    monkeypatch.setitem(base.CASES, name, BLOCKS[name])
    base.run_case(name, with_bwd=False)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("H,N,block", [(64, 2048, 512), (32, 3072, 768), (32, 4400, 1100), (32, 4096, 1024), (36, 4096, 2048)])
def test_many_heads_match_each_alone(H, N, block, D):
    """Tiles folded (2 and 4 to a block), numbered across all groups of an XCD and (D = 128, blocks of 2048) across eight and
    the one that is left: the same bits as head by head, far field included."""
    w = small("cfg2", D=D, N=N, Hq=H, Hkv=H, Cq=4, Ck=16, r=2, block=block, kmeans_iters=1)
    d = generate(w, need_dO=False)
    p = mb.params_for(w)
    Q, K, V = (d[x].to(p.torch_dtype).cuda().contiguous() for x in ("Q", "K", "V"))
    qc, qa, _, ka = mb.muse_cluster(p, Q, K, d["q_init_idx"].cuda(), d["k_init_idx"].cuda())
    O, LSE = mb.muse_fwd(p, Q, K, V, qc, qa, ka)[:2]
    one = mb.params_for(w, Hq=1, Hkv=1)
    for h in range(0, H, 13):
        part = [x[:, h:h + 1].contiguous() for x in (Q, K, V, qc, qa, ka)]
        a, b = mb.muse_fwd(one, *part)[:2]
        assert torch.equal(a, O[:, h:h + 1]) and torch.equal(b, LSE[:, h:h + 1])
