"""Queries and keys clustered in one call (two chains of launches on two streams) against each side alone: the same bits,
call after call on one workspace, with work queued before and behind the call on the caller's stream."""
import pytest
import torch

from paper_2509_10406_amd import binding as mb
from paper_2509_10406_amd.inputs import generate, small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,kw", [
    ("fp32", dict(N=2048, Cq=16, Ck=96, block=256)),
    ("bf16", dict(N=4096, Cq=48, Ck=200, block=512)),
    ("bf16", dict(N=4096, Cq=64, Ck=32, block=512, flags=mb.FLAG_STREAMING_KMEANS | mb.FLAG_BALANCED_ASSIGN)),
])
def test_both_sides_match_each_alone(dtype, kw):
    kw = dict(kw)
    flags = kw.pop("flags", 0)
    w = small("cfg1" if dtype == "fp32" else "cfg2", Hq=4, Hkv=2, r=1, **kw)
    d = generate(w, need_dO=False)
    p = mb.params_for(w, flags=flags)
    Q, K = (d[x].to(p.torch_dtype).cuda().contiguous() for x in ("Q", "K"))
    qi, ki = d["q_init_idx"].cuda(), d["k_init_idx"].cuda()
    for rep in range(4):
        alone = [t.clone() for t in mb.muse_cluster(p, Q, None, qi, None)[:2]]
        alone += [t.clone() for t in mb.muse_cluster(p, None, K, None, ki)[2:]]
        both = mb.muse_cluster(p, Q, K, qi, ki)
        Q.copy_(Q.flip(2)), K.copy_(K.flip(2))  # queued behind the call: must not reach it
        for a, b in zip(alone, both):
            assert torch.equal(a, b)
