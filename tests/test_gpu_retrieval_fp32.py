"""GPU parity of the fp32 backward where the retrieval's key/value gradients (retrieval_fp32.hip) tile keys by 16, queries
by 16 in pairs of tiles, and share a pair among hit slices.  Tolerance: the parity suite's 1e-4 of the largest entry."""
import pytest

import tests.test_gpu_muse as base

pytestmark = pytest.mark.gpu

CASES = {
    # some 40 keys per pair (three key tiles), two KV heads of two query heads each, heavy pairs (several slices)
    "fp32_pairs40": ("cfg1", dict(N=2048, Hq=4, Hkv=2, Cq=4, Ck=6, r=3, k2=2, block=256, kmeans_iters=1)),
    # every preceding block of one cluster: a pair's hits reach 448 x 1, no multiple of 32
    "fp32_all_blocks": ("cfg1", dict(N=960, Hq=2, Hkv=1, Cq=3, Ck=2, r=1, k2=0, block=120, kmeans_iters=1)),
    # the room of the partial rows: none for a second slice (one query head, one slot), room for two
    "fp32_one_slice": ("cfg1", dict(N=2048, Cq=2, Ck=2, r=1, block=256, kmeans_iters=1)),
    "fp32_two_slices": ("cfg1", dict(N=2048, Cq=2, Ck=3, r=2, block=256, kmeans_iters=1)),
    "fp32_d128": ("cfg1", dict(N=1024, D=128, Hq=2, Hkv=1, Cq=4, Ck=9, r=2, block=128, kmeans_iters=1)),
}
base.REACH.update({"fp32_pairs40": dict(pair_keys=33, pair_hits=512), "fp32_one_slice": dict(pair_hits=256),
                   "fp32_two_slices": dict(pair_hits=256)})


@pytest.mark.parametrize("name", list(CASES))
def test_fp32_retrieval_gradients(name, monkeypatch):
    monkeypatch.setitem(base.CASES, name, CASES[name])
    base.run_case(name, with_bwd=True)
