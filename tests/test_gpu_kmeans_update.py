"""GPU clustering where the centroid update and the fp32 assignment change their form: the wide and the narrow update on
clusters of every length (empty ones, one row, more than the rows in flight), more blocks than row slots, centroid
counts that fill no group of four.  The update must be the mean of the members (fp64, error of an fp32 sum of n terms: n
2^-24 times the mean absolute value), the assignment the nearest centroid wherever the margin is above 1e-5."""
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
