"""GPU parity of the far-field forward of bf16 inputs (k_farfield_tiles) where several waves share a tile of queries: every number
of tiles per wave at both head dimensions, waves that are left without a tile, lists of 8, 16 and 32 that are all selected, no
selection at all.  Scores that tie between waves, at the last place and in front of it.  The wide forms of large calls against
the narrow ones of single heads.  Tolerances are those of the parity suite.  And the weights of the softmax against 64 bits."""
import numpy as np
import pytest
import torch

import tests.test_gpu_muse as base
from paper_2509_10406_amd import binding as mb

pytestmark = pytest.mark.gpu

CASES = {f"waves_d{D}_ck{Ck}_r{r}": ("cfg2", dict(D=D, N=2048, Hq=2, Hkv=1, Cq=3, Ck=Ck, r=r, block=256, kmeans_iters=1))
         for D in (64, 128) for Ck, r in ((97, 8), (160, 32), (288, 16), (300, 0), (520, 4), (1030, 8), (1800, 32))}


@pytest.mark.parametrize("name", list(CASES))
def test_waves_of_a_tile(name, monkeypatch):
    monkeypatch.setitem(base.CASES, name, CASES[name])
    base.run_case(name, with_bwd=False)


@pytest.mark.parametrize("D,Ck,r,groups", [(64, 96, 8, 5), (64, 96, 5, 48), (128, 520, 16, 7), (64, 640, 32, 320), (128, 1100, 3, 1)])
def test_ties_between_waves(D, Ck, r, groups):
    """Key rows repeat with period `groups` inside a block and the key clusters hold one row each, so the clusters j, j + groups, ..
    of a block score the same to the last bit: of equal scores the lowest clusters are selected, and come first."""
    N, block = 8 * Ck, Ck
    g = torch.Generator().manual_seed(5)
    rows = torch.randn(groups, D, generator=g)
    K = rows[torch.arange(N) % block % groups].view(1, 1, N, D).bfloat16().cuda()
    Q, V = (torch.randn(1, 2, N, D, generator=g).bfloat16().cuda(), torch.randn(1, 1, N, D, generator=g).bfloat16().cuda())
    p = mb.Params(B=1, Hq=2, Hkv=1, N=N, D=D, Cq=4, Ck=Ck, r=r, k2=1, block=block, kmeans_iters=0, dtype=mb.BF16, grad_dtype=mb.FP32)
    qc = torch.randn(1, 2, 4, D, generator=g).cuda()
    aq = torch.randint(0, 4, (1, 2, N), generator=g, dtype=torch.int32).cuda()
    ak = (torch.arange(N, dtype=torch.int32) % block).view(1, 1, N).cuda()
    _, _, selc, _ = mb.muse_fwd(p, Q, K, V, qc, aq, ak)
    sel = selc.cpu().numpy()[0][:, block:]
    # score of cluster j: scale q.k_j of its row (the mass is the same for all): rank by the row, then by the cluster
    s = (Q[0, :, block:].double().cpu() @ rows.bfloat16().double().T).numpy()  # [2, far, groups]
    order = np.argsort(-s, axis=-1, kind="stable")
    top = np.sort(s, -1)[..., ::-1]
    members = [np.arange(x, Ck, groups) for x in range(groups)]
    sizes = np.array([len(m) for m in members])
    checked = 0
    for h in range(2):
        for n in range(0, sel.shape[1], 7):
            need = 1 + int(np.searchsorted(np.cumsum(sizes[order[h, n]]), r))  # rows that the selection reaches
            if groups > 1 and np.diff(-top[h, n, : need + 1]).min() < 1e-3 * np.abs(top[h, n]).max():
                continue  # two rows score nearly the same
            want = np.concatenate([members[x] for x in order[h, n, :need]])[:r]
            np.testing.assert_array_equal(sel[h, n], want)
            checked += 1
    assert checked > 100


@pytest.mark.parametrize("Ck,r", [(32, 4), (90, 8), (200, 16)])
def test_large_calls_as_single_heads(Ck, r):
    """Many heads have more tiles per wave than one head: the same scores, so the same selection; O up to the order of the sums."""
    N, D, H = 16384, 64, 32
    g = torch.Generator(device="cuda").manual_seed(3)
    Q, K, V = (torch.randn(1, H, N, D, generator=g, device="cuda").bfloat16() for _ in range(3))
    mk = lambda h: mb.Params(B=1, Hq=h, Hkv=h, N=N, D=D, Cq=16, Ck=Ck, r=r, k2=1, kmeans_iters=1, dtype=mb.BF16, grad_dtype=mb.FP32)
    init = lambda C: (torch.arange(C, device="cuda", dtype=torch.int32) * (N // C)).repeat(1, H, 1)
    qc, aq, _, ak = mb.muse_cluster(mk(H), Q, K, init(16), init(Ck))
    O, LSE, selc, selb = mb.muse_fwd(mk(H), Q, K, V, qc, aq, ak)
    for h in (0, 17, 31):
        one = [x[:, h : h + 1].contiguous() for x in (Q, K, V, qc, aq, ak)]
        o, lse, sc, sb = mb.muse_fwd(mk(1), *one)
        assert torch.equal(sc[0, 0], selc[0, h]) and torch.equal(sb[0, 0], selb[0, h])
        # fp32 sums in another order, then one bf16 rounding: one unit in the last place of the entry, or of the far field's share
        assert ((o[0, 0].float() - O[0, h].float()).abs() <= 2.0**-7 * O[0, h].float().abs() + 1e-4).all()
        torch.testing.assert_close(lse[0, 0], LSE[0, h], rtol=0, atol=1e-5)


@pytest.mark.parametrize("D,Ck,r", [(64, 40, 0), (64, 96, 1), (64, 300, 4), (64, 1100, 0), (128, 48, 3), (128, 300, 0), (128, 600, 16)])
def test_weights_against_64_bits(D, Ck, r):
    """With one key per cell the second block's queries attend the first block's keys exactly, by way of the summaries, and keys of their own
    block that weigh e^-64: O is the softmax's sum of the first block's values.  Its error is one rounding to bf16 (2^-9 of the
    entry) and what the weights' precision makes of sum p |v|: 2^-17 (a bf16 weight and a bf16 remainder) plus fp32 exponentials and
    scores (2^-18 for scores up to 16), bounded here at twice their sum.  Weights in bf16 alone are 2^-9 off."""
    g = torch.Generator().manual_seed(11)
    N, S = 2 * Ck, 1.0
    Q, K, V = (torch.randn(1, 1, N, D, generator=g) for _ in range(3))
    Q, K = Q * D**-0.5, K.clone()
    Q[..., 0], K[0, 0, :Ck, 0], K[0, 0, Ck:, 0] = 4.0, 0.0, -16.0
    Q, K, V = (x.bfloat16() for x in (Q, K, V))
    p = mb.Params(B=1, Hq=1, Hkv=1, N=N, D=D, Cq=3, Ck=Ck, r=r, k2=1, block=Ck, kmeans_iters=0, dtype=mb.BF16, grad_dtype=mb.FP32, scale=S)
    qc = 0.1 * torch.randn(1, 1, 3, D, generator=g)
    aq = torch.randint(0, 3, (1, 1, N), generator=g, dtype=torch.int32)
    ak = (torch.randperm(N, generator=g, dtype=torch.int32) % Ck).view(1, 1, N)
    ak[0, 0, :Ck] = torch.randperm(Ck, generator=g, dtype=torch.int32)
    O, LSE, _, _ = (x.cpu() for x in mb.muse_fwd(p, *(x.cuda() for x in (Q, K, V, qc, aq, ak))))
    q, k, v = (x[0, 0].double() for x in (Q, K, V))
    s = q[Ck:] @ k[:Ck].T
    w = s.softmax(-1)
    want = w @ v[:Ck]
    bound = 2.0**-8 * want.abs() + 2.0**-15 * (w @ v[:Ck].abs())
    err = (O[0, 0, Ck:].double() - want).abs()
    assert (err <= bound).all(), (err / bound).max()
    torch.testing.assert_close(LSE[0, 0, Ck:].double(), s.logsumexp(-1), rtol=0, atol=2e-5)
