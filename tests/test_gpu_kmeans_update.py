"""GPU clustering where the centroid update and the fp32 assignment change their form: centroid counts that fill no group of
four, clusters of every length (empty ones, one row, more than the rows in flight), more blocks than row slots.  Problems of
test_one_iteration's sizes take the update that reads the assignments; test_wide_and_narrow's take the two that walk the
buckets.  The update must be the mean of the members (fp64, error of an fp32 sum of n terms: n
2^-24 times the mean absolute value), the assignment the nearest centroid wherever the margin is above 1e-5."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle as orc
from paper_2509_10406_amd import binding as mb
from paper_2509_10406_amd.inputs import generate, small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("N,C,block", [(2048, 1, 128), (1536, 3, 96), (2048, 21, 256), (4096, 66, 512), (2048, 700, 256)])
def test_one_iteration(N, C, block, D, dtype):
    w = small("cfg1" if dtype == "fp32" else "cfg2", N=N, D=D, Hq=2, Hkv=2, Cq=C, Ck=C, r=1, block=block, kmeans_iters=1)
    d = generate(w, need_dO=False)
    p0, p1 = mb.params_for(w, kmeans_iters=0), mb.params_for(w)
    Q, K = (d[x].to(p0.torch_dtype).cuda().contiguous() for x in ("Q", "K"))
    qi, ki = d["q_init_idx"].cuda(), d["k_init_idx"].cuda()
    first = mb.muse_cluster(p0, Q, K, qi, ki)
    last = mb.muse_cluster(p1, Q, K, qi, ki)
    for X, c0, a0, c1, a1 in ((Q, first[0], first[1], last[0], last[1]), (K, first[2], first[3], last[2], last[3])):
        for h in range(2):
            x, a = X[0, h].double().cpu().numpy(), a0[0, h].cpu().numpy()
            for cent, assign in ((c0, a0), (c1, a1)):
                chk = orc.kmeans(x, C, 0, cent0=cent[0, h].double().cpu().numpy(), round_mode=int(dtype == "bf16"))
                safe = chk["margin"] > 1e-5
                np.testing.assert_array_equal(assign[0, h].cpu().numpy()[safe], chk["assign"][safe])
            n = np.bincount(a, minlength=C)
            tot, mag = np.zeros((C, D)), np.zeros((C, D))
            np.add.at(tot, a, x)
            np.add.at(mag, a, np.abs(x))
            want = np.where(n[:, None] > 0, tot / np.maximum(n, 1)[:, None], c0[0, h].double().cpu().numpy())
            bound = 2.0 ** -24 * np.maximum(n, 4)[:, None] * np.maximum(mag / np.maximum(n, 1)[:, None], np.abs(want))
            assert (np.abs(c1[0, h].double().cpu().numpy() - want) <= bound).all()


def form(H, N, C, D, dtype):
    """The launch's choice (kmeans.hip, scan_update and wide_update)."""
    S = 1024 // (D * (4 if dtype == "fp32" else 2))  # row slots
    if H * C * N <= 4 << 20 and N <= 8192 * S and H * C <= 2048 and H * C * S <= 8192:
        return "scan"
    return "wide" if (N // C // S >= 12 and H * C * S <= 8192) or N // C // S >= 64 else "narrow"


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("want_form,H,N,C,nb", [
    ("wide", 34, 16384, 8, 16),   # segments of some 128 rows, more blocks than slots
    ("wide", 2, 81920, 5, 10),    # few clusters of very many rows, blocks that fill no round of slots
    ("wide", 130, 8190, 5, 1),    # one block: one slot has everything
    ("narrow", 64, 1024, 66, 16),  # segments of one row and of none
    ("narrow", 90, 1500, 47, 12),
])
def test_wide_and_narrow(want_form, H, N, C, nb, D, dtype):
    assert form(H, N, C, D, dtype) == want_form
    g = torch.Generator(device="cuda").manual_seed(N + C)
    p1 = mb.Params(B=1, Hq=H, Hkv=H, N=N, D=D, Cq=C, Ck=C, block=N // nb, dtype=mb.FP32 if dtype == "fp32" else mb.BF16, kmeans_iters=1)
    p0 = dataclasses.replace(p1, kmeans_iters=0)
    X = torch.randn(1, H, N, D, generator=g, device="cuda").to(p1.torch_dtype)
    c0 = X[:, :, torch.randperm(N, generator=g, device="cuda")[:C]].float()
    c0[:, :, C // 2] = 100.0  # nobody's nearest: an empty cluster keeps its centroid
    a0 = mb.muse_cluster(p0, X, None, None, None, q_centroids=c0.clone())[1]
    c1 = mb.muse_cluster(p1, X, None, None, None, q_centroids=c0.clone())[0]
    for h in (0, H // 2, H - 1):
        x, a = X[0, h].double().cpu().numpy(), a0[0, h].cpu().numpy()
        n = np.bincount(a, minlength=C)
        assert n[C // 2] == 0
        tot, mag = np.zeros((C, D)), np.zeros((C, D))
        np.add.at(tot, a, x)
        np.add.at(mag, a, np.abs(x))
        want = np.where(n[:, None] > 0, tot / np.maximum(n, 1)[:, None], c0[0, h].double().cpu().numpy())
        bound = 2.0 ** -24 * np.maximum(n, 4)[:, None] * np.maximum(mag / np.maximum(n, 1)[:, None], np.abs(want))
        assert (np.abs(c1[0, h].double().cpu().numpy() - want) <= bound).all()
