"""dQ, dK and dV of bf16 attention in tiles of 256 rows, where those tiles end: a block of one tile and a row more, last tiles with
one row, with one wave, with an odd half of a wave's 64 (D = 128: tiles of 128 keys, seeds in chunks of 256 rows), blocks of whole tiles, grouped query heads (their steps follow one another),
and enough heads that dQ takes these tiles too.  Against fp64 on the same bf16 rows, entry by entry at the rounding of the operands;
several blocks and sequences against one block at a time; rows that are not finite."""
import math

import pytest
import torch

from paper_2509_10406_amd import binding as mb

pytestmark = pytest.mark.gpu


def _head(q, k, v, d, o, lse, scale):
    """dQ, dK, dV of one head in 64 bits at the O and LSE that the call was given, each with a bound for every entry: P (in dV) and
    dS (in dQ and dK) enter their products as bf16 (8 significant bits, to nearest: 2^-8 of each), the
    products are added in fp32 (here at most a tenth of that), and dS inherits the fp32 sums dP and dO.O (2^-16 of the sums of the sizes)."""
    P = (q @ k.T * scale - lse[:, None]).exp().tril()
    dP, delta = d @ v.T, (d * o).sum(-1, keepdim=True)
    dS = P * (dP - delta)
    eS = 1.1 * 2.0 ** -8 * dS.abs() + 2.0 ** -16 * P * (d.abs() @ v.abs().T + (d * o).abs().sum(-1, keepdim=True))
    return ((scale * dS @ k, scale * eS @ k.abs()), (scale * dS.T @ q, scale * eS.T @ q.abs()),
            (P.T @ d, 1.1 * 2.0 ** -8 * P.T @ d.abs()))


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

    def check(x, want, bound, first, what):
        over = (x.double() - want).abs() - bound
        assert over.max() <= 0, (what, divmod(int(over.argmax()), D), float(over.max()))
        # a row left out or taken from elsewhere would be seen: it is larger than its bound (the first dQ row is zero but for rounding)
        assert (want.abs() > bound).any(-1)[first:].all(), what

    for hk in range(Hkv):
        k, v = K[0, hk].double(), V[0, hk].double()
        sums = [torch.zeros_like(k) for _ in range(4)]
        for h in range(hk * G, hk * G + G):
            (wq, bq), wk, wv = _head(Q[0, h].double(), k, v, dO[0, h].double(), O[0, h].double(), LSE[0, h].double(), 1 / math.sqrt(D))
            check(got[0][0, h], wq, bq, 1, f"dQ {h}")
            for s, x in zip(sums, (*wk, *wv)):
                s += x
        check(got[1][0, hk], sums[0], sums[1], 0, f"dK {hk}")
        check(got[2][0, hk], sums[2], sums[3], 0, f"dV {hk}")


@pytest.mark.parametrize("D", [64, 128])
def test_blocks_and_sequences(D):
    # several blocks that end inside a tile, two sequences, grouped heads, more groups than an XCD takes at a time and a last turn with
    # fewer: every block has the bits of exact attention over its own rows.  Rows of different blocks are so far apart (128 in the
    # logit) that the far field is zero in fp32.
    g = torch.Generator().manual_seed(D)
    B, Hq, Hkv, Bs, nb = 2, 40, 20, 1100, 3
    N = Bs * nb
    Q, K, V, dO = (torch.randn(B, H, N, D, generator=g) for H in (Hq, Hkv, Hkv, Hq))
    for b in range(nb):
        for x in (Q, K):
            x[:, :, :, b] = 0
            x[:, :, b * Bs:(b + 1) * Bs, b] = 32
    Q, K, V, dO = (x.bfloat16().cuda() for x in (Q, K, V, dO))
    p = mb.Params(B=B, Hq=Hq, Hkv=Hkv, N=N, D=D, Cq=1, Ck=1, block=Bs, scale=0.125)
    qc = Q.float().mean(2, keepdim=True).contiguous()
    qa, ka = (torch.zeros(B, H, N, dtype=torch.int32, device="cuda") for H in (Hq, Hkv))
    O, LSE, selc, selb = mb.muse_fwd(p, Q, K, V, qc, qa, ka)
    got = mb.muse_bwd(p, Q, K, V, O, LSE, dO, qc, qa, ka, selc, selb)
    pb = mb.Params(B=B, Hq=Hq, Hkv=Hkv, N=Bs, D=D, scale=0.125)
    for b in range(nb):
        at = slice(b * Bs, (b + 1) * Bs)
        q, k, v, o, l, d = (x[:, :, at].contiguous() for x in (Q, K, V, O, LSE, dO))
        for what, x, y in zip(("dQ", "dK", "dV"), got, mb.exact_attn_bwd(pb, q, k, v, o, l, d)):
            assert torch.equal(x[:, :, at], y), (what, b)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("n", [650, 700])
@pytest.mark.parametrize("what", ["Q", "K", "V", "dO"])
def test_where_a_row_that_is_not_finite_goes(what, n, D):
    # a pair that the mask removes is still met inside the 32 x 32 square on the diagonal, and nowhere else.  A row of Q or dO reaches
    # its own dQ and the keys up to the end of that square, a row of K or V the queries from the square's first on.
    g = torch.Generator().manual_seed(6)
    H, N = 32, 1100
    p = mb.Params(B=1, Hq=H, Hkv=H, N=N, D=D)
    t = {x: torch.randn(1, H, N, D, generator=g).bfloat16().cuda() for x in ("Q", "K", "V", "dO")}
    O, LSE = mb.exact_attn_fwd(p, t["Q"], t["K"], t["V"])
    want = mb.exact_attn_bwd(p, t["Q"], t["K"], t["V"], O, LSE, t["dO"])
    t[what][:, ::2, n, 3], t[what][:, 1::2, n, 3] = float("inf"), float("nan")
    dQ, dK, dV = mb.exact_attn_bwd(p, t["Q"], t["K"], t["V"], O, LSE, t["dO"])
    rows, square = torch.arange(N, device="cuda"), n // 32 * 32
    if what in ("Q", "dO"):
        others, later = rows != n, rows >= square + 32
        assert torch.equal(dQ[:, :, others], want[0][:, :, others])
        assert torch.equal(dK[:, :, later], want[1][:, :, later]) and torch.equal(dV[:, :, later], want[2][:, :, later])
        assert not dQ[:, :, n].isfinite().all(-1).any()
    else:
        earlier = rows < square
        assert torch.equal(dQ[:, :, earlier], want[0][:, :, earlier])
        assert not dQ[:, :, n].isfinite().all(-1).any()


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
