"""A query row of Q or dO that is not finite (an overflow one wants to find) reaches the gradients of the keys that the query
attends, directly or through a summary, and nothing behind its own block: the keys of later blocks get what they get without
that row, and the other queries' dQ is untouched.  Clusters of many queries, so that the chains' tiles mix blocks.  In the forward
without retrieval, cluster scores that overflow reach that query's output, and no other query's."""
import math

import pytest
import torch

from paper_2509_10406_amd import binding as mb
from paper_2509_10406_amd.inputs import generate, small
from tests.util import BF16_ABS, FP32_REL

pytestmark = pytest.mark.gpu

CASES = {
    "fp32": ("cfg1", dict(N=1024, Cq=2, Ck=6, r=2, block=128, kmeans_iters=2)),
    "fp32_nb16_d128": ("cfg1", dict(N=1024, D=128, Hq=2, Hkv=1, Cq=2, Ck=6, r=3, k2=2, block=64, kmeans_iters=2)),
    "bf16": ("cfg2", dict(N=1024, Hq=2, Hkv=1, Cq=2, Ck=6, r=2, block=128, kmeans_iters=2)),
    "bf16_nb16": ("cfg2", dict(N=1024, Hq=1, Hkv=1, Cq=1, Ck=5, r=2, block=64, kmeans_iters=2)),
    "bf16_d128": ("cfg5", dict(N=1024, Hq=1, Hkv=1, Cq=2, Ck=6, r=2, block=128, kmeans_iters=2)),
}


@pytest.mark.parametrize("what", ["dO", "Q"])
@pytest.mark.parametrize("name", list(CASES))
def test_rows_that_are_not_finite_stay_in_their_past(name, what):
    base, kw = CASES[name]
    w = small(base, **kw)
    d = generate(w, need_dO=True)
    p = mb.params_for(w)
    Q, K, V, dO = (d[x].to(p.torch_dtype).cuda().contiguous() for x in ("Q", "K", "V", "dO"))
    qc, qa, _, ka = mb.muse_cluster(p, Q, K, d["q_init_idx"].cuda(), d["k_init_idx"].cuda())
    O, LSE, selc, selb = mb.muse_fwd(p, Q, K, V, qc, qa, ka)
    for n in range(2 * w.Bs + 5, w.N - w.Bs, w.N // 6):
        without, Qi, gi = dO.clone(), Q.clone(), dO.clone()
        without[0, 0, n] = 0.0
        (gi if what == "dO" else Qi)[0, 0, n] = math.inf
        Oi, Li = O.clone(), LSE.clone()
        if what == "Q":                               # the forward of such a row has given no number
            Oi[0, 0, n], Li[0, 0, n] = math.nan, math.nan
        want = mb.muse_bwd(p, Q, K, V, O, LSE, without, qc, qa, ka, selc, selb)
        got = mb.muse_bwd(p, Qi, K, V, Oi, Li, gi, qc, qa, ka, selc, selb)
        later = (n // w.Bs + 1) * w.Bs
        for i in (1, 2):
            a, b = got[i][:, :, later:].double(), want[i][:, :, later:].double()
            tol = FP32_REL * float(want[i].abs().max()) if p.dtype == mb.FP32 else BF16_ABS
            assert a.isfinite().all() and (a - b).abs().max() <= tol, ("dK", "dV")[i - 1]
        others = torch.ones(w.N, dtype=torch.bool)
        others[n] = False
        assert got[0][0, 0, others].isfinite().all() and not got[0][0, 0, n].isfinite().all()
        assert not got[1][0, 0, : n + 1].isfinite().all()


@pytest.mark.parametrize("D,Ck", [(64, 40), (64, 300), (128, 40), (128, 600)])
def test_overflowing_scores_reach_the_output(D, Ck):
    """A finite query row with one entry past the fp16 range has infinite scores, of both signs, against the remainder plane of the
    key summaries.  With nothing retrieved their softmax is no number, and must not come out as the softmax of the rest; the
    other rows keep their bits."""
    N, block, n = 16 * Ck, 2 * Ck, 15 * Ck + 3
    g = torch.Generator(device="cuda").manual_seed(7)
    Q, K, V = (torch.randn(1, 1, N, D, generator=g, device="cuda").bfloat16() for _ in range(3))
    p = mb.Params(B=1, Hq=1, Hkv=1, N=N, D=D, Cq=2, Ck=Ck, r=0, k2=1, block=block, kmeans_iters=0, dtype=mb.BF16, grad_dtype=mb.FP32)
    qc = torch.randn(1, 1, 2, D, generator=g, device="cuda")
    aq = torch.randint(0, 2, (1, 1, N), generator=g, device="cuda", dtype=torch.int32)
    ak = (torch.arange(N, device="cuda", dtype=torch.int32) % Ck).view(1, 1, N)  # two keys a cell: no summary is a bf16 row
    O, LSE, _, _ = mb.muse_fwd(p, Q, K, V, qc, aq, ak)
    Qi = Q.clone()
    Qi[0, 0, n, 3] = 80000.0
    Oi, Li, _, _ = mb.muse_fwd(p, Qi, K, V, qc, aq, ak)
    others = torch.arange(N, device="cuda") != n
    assert O.isfinite().all() and torch.equal(Oi[0, 0, others], O[0, 0, others]) and torch.equal(Li[0, 0, others], LSE[0, 0, others])
    assert not Li[0, 0, n].isfinite() and not Oi[0, 0, n].isfinite().any()
