"""Many short sequences in one call: the heads of queries and keys together are more than a launch takes in one dimension of its grid,
those of either side are not.  The call is accepted and gives every sequence what a call of its own gives it."""
import pytest
import torch

from paper_2509_10406_amd import binding as mb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [mb.BF16, mb.FP32])
def test_heads_of_both_sides_beyond_one_grid(dtype):
    B, N, C = 33000, 32, 2  # 66000 heads of queries and keys
    g = torch.Generator(device="cuda").manual_seed(5)
    p = mb.Params(B=B, Hq=1, Hkv=1, N=N, D=64, Cq=C, Ck=C, r=1, k2=1, block=N // 2, kmeans_iters=1, dtype=dtype)
    Q, K, V = (torch.randn(B, 1, N, 64, generator=g, device="cuda").to(p.torch_dtype) for _ in range(3))
    init = torch.tensor([3, 20], dtype=torch.int32, device="cuda").repeat(B, 1, 1)
    qc, aq, kc, ak = mb.muse_cluster(p, Q, K, init, init)
    got = mb.muse_fwd(p, Q, K, V, qc, aq, ak)
    for lo, hi in ((0, 100), (B // 2 - 50, B // 2 + 50), (B - 100, B)):
        q = mb.Params(**{**p.__dict__, "B": hi - lo})
        one = [x[lo:hi].contiguous() for x in (Q, K, V, init)]
        c = mb.muse_cluster(q, one[0], one[1], one[3], one[3])
        assert all(torch.equal(a, b[lo:hi]) for a, b in zip(c, (qc, aq, kc, ak)))
        for a, b in zip(mb.muse_fwd(q, *one[:3], c[0], c[1], c[3]), got):
            torch.testing.assert_close(a, b[lo:hi], rtol=2.0**-7 if dtype == mb.BF16 else 1e-5, atol=1e-5)
    mb.free_workspaces()
