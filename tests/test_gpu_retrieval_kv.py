"""GPU parity of the bf16 retrieval where its kernels change form.  Query side (retrieval_q.hip): 64 keys staged at a time,
so pairs of up to 64 keys and of several stages.  Key/value gradients (retrieval_kv.hip): pairs of up to
32 keys (the waves share the hits), 33 to 64 (a wave per key tile) and more (several key groups), several hit slices, one
hit, and grouped queries.  D = 128 with several key groups is bf16_d128_pairs40 of the parity suite (more keys per pair
than its 40 put the query gradient, another kernel's, at its bound of 2e-2).  Tolerance: the parity suite's."""
import pytest

import tests.test_gpu_muse as base

pytestmark = pytest.mark.gpu

CASES = {
    "kv_pairs40_gqa": ("cfg2", dict(N=2048, Hq=4, Hkv=2, Cq=4, Ck=6, r=3, k2=2, block=256, kmeans_iters=1)),
    "kv_pairs250": ("cfg2", dict(N=4096, Hq=2, Hkv=1, Cq=3, Ck=2, r=1, block=512, kmeans_iters=1)),
    "kv_single_hits": ("cfg2", dict(N=512, Hq=1, Hkv=1, Cq=8, Ck=60, r=1, block=64, kmeans_iters=1)),
}
base.REACH.update({"kv_pairs40_gqa": dict(pair_keys=33, pair_hits=512), "kv_pairs250": dict(pair_keys=129, pair_hits=512)})


@pytest.mark.parametrize("name", list(CASES))
def test_retrieval_key_value_gradients(name, monkeypatch):
    monkeypatch.setitem(base.CASES, name, CASES[name])
    base.run_case(name, with_bwd=True)
