"""GPU parity of the backward where component 2 of the cell gradients (chain_grads.hip) changes its path: chunks of a
query cluster, chains per workgroup (waves that share a chain, pairs of chains, an odd chain left over), more than eight
preceding key blocks, both head dimensions and both input types.  Tolerances are those of the parity suite."""
import pytest

import tests.test_gpu_muse as base

pytestmark = pytest.mark.gpu

CASES = {
    # a cluster of 1536 far-field queries: three chunks of 512; one chain, shared by four waves
    "chains_1x1536": ("cfg2", dict(N=2048, Hq=1, Hkv=1, Cq=1, Ck=1, r=1, block=512, kmeans_iters=1)),
    # r = 20: chunks of 204 queries (list capacity), nearly every chain retrieved by nearly every query
    "chains_r20": ("cfg2", dict(N=1024, Hq=1, Hkv=1, Cq=1, Ck=24, r=20, block=256, kmeans_iters=1)),
    # a grid that needs no spreading: all chains of a word in one workgroup, odd counts among them
    "chains_word": ("cfg2", dict(N=2048, Hq=8, Hkv=8, Cq=256, Ck=40, r=4, block=256, kmeans_iters=1)),
    # eight chains of a word per workgroup
    "chains_quarter": ("cfg2", dict(N=2048, Hq=8, Hkv=4, Cq=64, Ck=32, r=5, k2=2, block=256, kmeans_iters=1)),
    "chains_d128_nb12": ("cfg5", dict(N=1536, Hq=2, Hkv=1, Cq=2, Ck=35, r=9, block=128, kmeans_iters=1)),
    "chains_d128_word": ("cfg2", dict(D=128, N=1024, Hq=8, Hkv=2, Cq=128, Ck=64, r=3, block=128, kmeans_iters=1)),
    "chains_fp32": ("cfg1", dict(N=1536, Cq=1, Ck=7, r=3, block=192, kmeans_iters=1)),
    "chains_fp32_nb16": ("cfg1", dict(N=1024, Cq=3, Ck=33, r=5, block=64, kmeans_iters=1)),
    "chains_fp32_d128": ("cfg1", dict(N=1024, Hq=2, Hkv=2, D=128, Cq=64, Ck=48, r=4, block=128, kmeans_iters=1)),
}

# rotary rows: entries of dQ at up to 2.6e-2 against gradients at the exact O, where the suite's bound is 2.2e-2 (a bf16 unit
# of the largest entry); at the O that the library is handed 2.3e-2, inside what the rounding of the operands gives
OWN_OUTPUTS = {
    "chains_d128_word_rotary": ("cfg5", dict(N=1024, Hq=8, Hkv=2, Cq=128, Ck=64, r=3, block=128, kmeans_iters=1)),
}


@pytest.mark.parametrize("name", list(OWN_OUTPUTS))
def test_chain_gradients_of_rotary_rows(name, monkeypatch):
    monkeypatch.setitem(base.CASES, name, OWN_OUTPUTS[name])
    base.run_case(name, with_bwd=True, own_outputs=True)


@pytest.mark.parametrize("name", list(CASES))
def test_chain_gradients(name, monkeypatch):
    monkeypatch.setitem(base.CASES, name, CASES[name])
    base.run_case(name, with_bwd=True)
