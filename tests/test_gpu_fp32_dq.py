"""GPU parity of the fp32 backward where the per-query walk of dQ (component 2 and the retrieved keys) changes its path: no
key, fewer keys than are requested together and not a multiple of them, every preceding block retrieved, more than eight key
blocks, more than eight and sixteen slots.  Tolerances are those of the parity suite."""
import pytest

import tests.test_gpu_muse as base

pytestmark = pytest.mark.gpu

CASES = {
    "f32dq_few_keys": ("cfg1", dict(N=512, Hq=2, Hkv=1, Cq=4, Ck=40, r=6, block=64, kmeans_iters=1)),
    "f32dq_many_keys": ("cfg1", dict(N=768, Hq=1, Hkv=1, Cq=2, Ck=3, r=2, k2=2, block=192, kmeans_iters=1)),
    "f32dq_all_blocks": ("cfg1", dict(N=512, Hq=1, Hkv=1, Cq=4, Ck=12, r=4, k2=0, block=128, kmeans_iters=1)),
    "f32dq_nb16_r17": ("cfg1", dict(N=1024, Hq=2, Hkv=2, Cq=4, Ck=33, r=17, block=64, kmeans_iters=1)),
    "f32dq_d128_r9": ("cfg1", dict(D=128, N=512, Hq=2, Hkv=1, Cq=4, Ck=20, r=9, k2=2, block=64, kmeans_iters=1)),
    "selinfo_r32": ("cfg2", dict(N=512, Hq=1, Hkv=1, Cq=4, Ck=40, r=32, k2=2, block=64, kmeans_iters=1)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_fp32_dq(name, monkeypatch):
    monkeypatch.setitem(base.CASES, name, CASES[name])
    base.run_case(name, with_bwd=True)
