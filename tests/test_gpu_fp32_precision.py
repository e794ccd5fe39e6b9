"""fp32 scores come from sums of 16 products, not from one chain of D: what a score is off by, its whole softmax row is.
A chain of n products with random signs rounds by some sqrt(n / 2) 2^-24 of its rms; 16 products and the D / 16 partial
sums give 2.2 to 2.4 times sqrt(D) |q k| 2^-24, one chain of D 5.7 (D = 64) to 8 (D = 128).  The bounds, on the norm against
64 bits, are 1.3 to 1.6 times what sums of 16 show; one chain is above them."""
import math

import numpy as np
import pytest
import torch

import oracle as orc
from paper_2509_10406_amd import binding as mb
from paper_2509_10406_amd.inputs import generate, small
from tests.util import f64, oracle_head

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,most", [(64, (6.5e-7, 1.6e-6, 1.6e-6)), (128, (7.0e-7, 1.8e-6, 1.8e-6))])
def test_scores_of_peaked_rows(D, most):
    """Rows three times as large as usual: logits up to some 30, where the error of a score shows most."""
    g = torch.Generator(device="cuda").manual_seed(D)
    N = 1024
    p = mb.Params(B=1, Hq=2, Hkv=1, N=N, D=D, dtype=mb.FP32, grad_dtype=mb.FP32)
    Q, K, V, dO = (3.0 * torch.randn(1, h, N, D, generator=g, device="cuda") for h in (2, 1, 1, 2))
    O, LSE = mb.exact_attn_fwd(p, Q, K, V)
    dQ, dK, _ = mb.exact_attn_bwd(p, Q, K, V, O, LSE, dO)
    q, k, v = (x.double().requires_grad_() for x in (Q, K, V))
    S = (q @ k.transpose(-1, -2)) / math.sqrt(D)
    want = S.masked_fill(torch.ones(N, N, dtype=torch.bool, device="cuda").triu(1), -math.inf).softmax(-1) @ v
    want.backward(dO.double())
    for what, a, b, bound in (("O", O, want.detach(), most[0]), ("dQ", dQ, q.grad, most[1]), ("dK", dK, k.grad, most[2])):
        err = ((a.double() - b).norm() / b.norm()).item()
        print(f"{what} D={D}: {err:.2e} (bound {bound:.1e})")
        assert err <= bound, (what, err)


def test_summaries_and_retrieval_of_rotary_rows():
    """dK and dV of the whole layer at D = 128: chains of summaries and retrieved pairs (rotary rows, logits up to some 10)."""
    w = small("cfg5", N=1024, Hq=1, Hkv=1, Cq=8, Ck=24, r=4, block=128, kmeans_iters=2, dtype="fp32")
    d = generate(w, need_dO=True)
    p = mb.params_for(w)
    Q, K, V, dO = (d[x].cuda().contiguous() for x in ("Q", "K", "V", "dO"))
    qc, qa, _, ka = mb.muse_cluster(p, Q, K, d["q_init_idx"].cuda(), d["k_init_idx"].cuda())
    O, LSE, selc, selb = mb.muse_fwd(p, Q, K, V, qc, qa, ka)
    got = mb.muse_bwd(p, Q, K, V, O, LSE, dO, qc, qa, ka, selc, selb)
    op = orc.MuseParams(w.N, w.D, w.Bs, w.Cq, w.Ck, w.r, w.k2, p.eff_scale)
    sel = (selc.cpu().numpy()[0, 0], selb.cpu().numpy()[0, 0].reshape(w.N, w.r, op.k2e))
    want = oracle_head(orc, op, *(f64(x[0, 0]) for x in (Q, K, V, dO)), f64(qc[0, 0]), qa[0, 0].cpu().numpy(), ka[0, 0].cpu().numpy(), sel)["grads"]
    for what, a, b in zip(("dQ", "dK", "dV"), got, want):
        err = np.linalg.norm(f64(a[0, 0]) - b) / np.linalg.norm(b)
        print(f"{what}: {err:.2e}")
        assert err <= (9e-7 if what == "dQ" else 7e-7), (what, err)
