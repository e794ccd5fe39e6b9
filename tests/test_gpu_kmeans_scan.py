"""The centroid update that finds its members in the assignments themselves (small problems) at the sizes where it can go
wrong: blocks of odd length and of more positions than a scan step, empty clusters, more blocks than row slots, lists of
more than 64 members.  One update from random centroids against the mean of the members in fp64: the error of an fp32 sum
of n terms, n 2^-24 times the mean absolute value."""
import numpy as np
import pytest
import torch

from paper_2509_10406_amd import binding as mb
from tests.test_gpu_kmeans_update import form

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [mb.FP32, mb.BF16])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("N,nb,C", [(749 * 8, 8, 23), (2048, 16, 3), (4100, 2, 40), (7, 7, 5), (8192, 1, 1), (1536, 12, 130)])
def test_update_from_assignments(N, nb, C, D, dtype):
    g = torch.Generator().manual_seed(N + C + D)
    X = torch.randn(1, 2, N, D, generator=g)
    X[:, 1] *= 0.1
    cent = X[:, :, torch.randperm(N, generator=g)[:C]].clone()
    if C > 4:
        cent[:, :, 3] = 100.0  # nobody's nearest: keeps its centroid
    p = mb.Params(B=1, Hq=2, Hkv=2, N=N, D=D, Cq=C, Ck=C, block=N // nb, dtype=dtype, kmeans_iters=1)
    Xd = X.to(p.torch_dtype).cuda()
    assert form(2, N, C, D, "fp32" if dtype == mb.FP32 else "bf16") == "scan"
    import dataclasses
    c0 = cent.cuda()
    a0 = mb.muse_cluster(dataclasses.replace(p, kmeans_iters=0), Xd, None, None, None, q_centroids=c0.clone())[1]
    c1 = mb.muse_cluster(p, Xd, None, None, None, q_centroids=c0.clone())[0]
    for h in range(2):
        x, a = Xd[0, h].double().cpu().numpy(), a0[0, h].cpu().numpy()
        n = np.bincount(a, minlength=C)
        tot, mag = np.zeros((C, D)), np.zeros((C, D))
        np.add.at(tot, a, x)
        np.add.at(mag, a, np.abs(x))
        want = np.where(n[:, None] > 0, tot / np.maximum(n, 1)[:, None], cent[0, h].double().numpy())
        bound = 2.0 ** -24 * np.maximum(n, 4)[:, None] * np.maximum(mag / np.maximum(n, 1)[:, None], np.abs(want))
        assert (np.abs(c1[0, h].double().cpu().numpy() - want) <= bound).all()
