"""GPU parity of the kernels that take the far-field queries one by one (component 2, forward and dQ) at odd counts: clusters that no
query is in, two, three, nine (a second chunk of eight key blocks) and sixteen blocks, ends of the order that fill no workgroup and rounds of
workgroups that are not full.  Tolerances are those of the parity suite."""
import pytest

import tests.test_gpu_muse as base

pytestmark = pytest.mark.gpu

CASES = {
    "fq_cq16_nb2": ("cfg2", dict(N=272, Hq=1, Hkv=1, Cq=16, Ck=24, r=3, block=136, kmeans_iters=1)),
    "fq_cq7_nb3": ("cfg2", dict(N=603, Hq=2, Hkv=1, Cq=7, Ck=19, r=3, block=201, kmeans_iters=1)),
    "fq_cq7_nb3_k2_2": ("cfg5", dict(N=402, Hq=2, Hkv=1, Cq=7, Ck=11, r=11, k2=2, block=134, kmeans_iters=1)),
    "fq_cq17_nb10": ("cfg2", dict(N=1030, Hq=2, Hkv=1, Cq=17, Ck=33, r=4, k2=2, block=103, kmeans_iters=1)),
    "fq_cq300_nb8": ("cfg2", dict(N=2048, Hq=2, Hkv=1, Cq=300, Ck=40, r=4, block=256, kmeans_iters=1)),
    "fq_cq257_nb16": ("cfg2", dict(N=2048, Hq=1, Hkv=1, Cq=257, Ck=30, r=9, k2=3, block=128, kmeans_iters=1)),
    "fq_fp32_cq300": ("cfg1", dict(N=2048, Cq=300, Ck=40, r=4, block=256, kmeans_iters=1)),
    "fq_fp32_nb3": ("cfg1", dict(N=603, Cq=7, Ck=19, r=3, block=201, kmeans_iters=1)),
    "fq_fp32_nb10": ("cfg1", dict(N=1030, Cq=17, Ck=33, r=4, k2=2, block=103, kmeans_iters=1)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_far_queries(name, monkeypatch):
    monkeypatch.setitem(base.CASES, name, CASES[name])
    base.run_case(name, with_bwd=True)
