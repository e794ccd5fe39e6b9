"""Rows of Q or K with a NaN or an infinity in them (an overflow one wants to find): they get a cluster number that exists, and
the same one whichever form of the centroid update runs."""
import dataclasses
import math

import pytest
import torch

from paper_2509_10406_amd import binding as mb
from tests.test_gpu_kmeans_update import form

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bad", [math.nan, math.inf, -math.inf])
@pytest.mark.parametrize("D,C", [(64, 70), (128, 70), (64, 520)])
def test_lloyd(D, C, bad):
    N = 1024
    g = torch.Generator().manual_seed(D + C)
    X = torch.randn(1, 1, N, D, generator=g)
    X[0, 0, 5], X[0, 0, 700, 3] = bad, bad
    at = torch.randperm(N - 6, generator=g)[:C] + 6
    at[at == 700] = 6
    got = []
    # one head: the update that reads the assignments; many: the one behind the bucketing
    for H in (1, 96):
        assert (form(H, N, C, D, "bf16") == "scan") == (H == 1)
        p = mb.Params(B=1, Hq=H, Hkv=H, N=N, D=D, Cq=C, Ck=C, kmeans_iters=3)
        x, init = X.expand(1, H, N, D).bfloat16().cuda().contiguous(), at.int().expand(1, H, C).cuda().contiguous()
        cent, assign = mb.muse_cluster(p, x, None, init, None)[:2]
        assert int(assign.min()) >= 0 and int(assign.max()) < C
        a = assign.cpu()
        if C < 480:  # no score at all (past 480 an infinite one can be kept): both rows are the last cluster's, nobody else's
            assert (a[..., [5, 700]] == C - 1).all()
            assert (cent.isfinite().all(-1).sum(-1) == C - 1).all() and cent[:, :, : C - 1].isfinite().all()
        assert (a == a[:, :1]).all() and torch.equal(cent.nan_to_num(), cent[:, :1].nan_to_num().expand_as(cent))
        got.append((cent[:, 0].cpu(), a[:, 0]))
    assert torch.equal(got[0][1], got[1][1]) and torch.equal(got[0][0].nan_to_num(), got[1][0].nan_to_num())


@pytest.mark.parametrize("dtype", [mb.FP32, mb.BF16])
@pytest.mark.parametrize("bad", [math.nan, math.inf, 1e30])  # the pass runs in binary16
@pytest.mark.parametrize("D,C", [(64, 3), (128, 70), (64, 1030)])  # few: the state in LDS
def test_streaming(D, C, bad, dtype):
    N = 2080
    g = torch.Generator().manual_seed(D + C)
    X = torch.randn(1, 2, N, D, generator=g)
    X[0, 0, 1500], X[0, 0, 2000, 3] = bad, bad
    at = torch.stack([torch.randperm(1400, generator=g)[:C] for _ in range(2)]).int()[None].cuda()
    p = mb.Params(B=1, Hq=2, Hkv=2, N=N, D=D, Cq=C, Ck=C, dtype=dtype)
    x = X.to(p.torch_dtype).cuda()
    cent, assign, counts = mb.muse_kmeans_stream(p, 0, x, at)
    assert int(assign.min()) >= 0 and int(assign.max()) < C and counts.isfinite().all()
    assert cent[0, 1].isfinite().all()  # the other head
    if C > 3:  # two rows spoil two centroids at most
        assert int((~cent[0, 0].isfinite().all(-1)).sum()) in (1, 2)
    final = mb.muse_cluster(dataclasses.replace(p, flags=mb.FLAG_STREAMING_KMEANS), x, None, at, None)[1]
    assert int(final.min()) >= 0 and int(final.max()) < C
