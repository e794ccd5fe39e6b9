"""GPU parity of the backward of bf16 inputs where the lists behind component 2 of the cell gradients (k_chain_lists, k_chain_grads)
change their form: one, several and no whole 64 queries per wave, slots loaded four at a time and one by one, numbers of
clusters of 5 to 11 bits, one-wave workgroups that loop over a cluster's chains, waves that share a chain.  Tolerances are those
of the parity suite.  And several backwards on one kept state, the first of which writes the lists over the forward's."""
import dataclasses

import pytest
import torch

import tests.test_gpu_muse as base
from paper_2509_10406_amd import binding as mb
from paper_2509_10406_amd.inputs import generate, small

pytestmark = pytest.mark.gpu

CASES = {
    # one-wave workgroups, more than 128 chains of a cluster: a wave takes several pairs
    "lists_many_chains": ("cfg2", dict(N=2048, Hq=8, Hkv=4, Cq=32, Ck=300, r=16, block=256, kmeans_iters=1)),
    # 11 bits, slots one by one, more than eight of them
    "lists_bits11": ("cfg2", dict(N=2048, Hq=2, Hkv=1, Cq=4, Ck=1100, r=9, block=256, kmeans_iters=1)),
    "lists_bits10_d128": ("cfg2", dict(D=128, N=2048, Hq=2, Hkv=2, Cq=4, Ck=520, r=12, block=256, kmeans_iters=1)),
    # eight waves per cluster: 600 clusters of some 500 queries
    "lists_8_waves": ("cfg2", dict(N=4096, Hq=75, Hkv=75, Cq=8, Ck=20, r=3, block=512, kmeans_iters=1)),
    # four waves, blocks beyond nine
    "lists_nb16": ("cfg2", dict(N=2048, Hq=40, Hkv=20, Cq=16, Ck=33, r=6, k2=2, block=128, kmeans_iters=1)),
    # a cluster of 3584 far queries: several rounds of 64 per wave
    "lists_one_cluster": ("cfg2", dict(N=4096, Hq=1, Hkv=1, Cq=1, Ck=40, r=20, block=512, kmeans_iters=1)),
    # few query clusters: every group of chains has a workgroup of its own, whose waves share it; one and two chains a group
    "lists_shared_nb16": ("cfg2", dict(N=2048, Hq=2, Hkv=1, Cq=2, Ck=37, r=6, k2=2, block=128, kmeans_iters=1)),
    "lists_shared_d128": ("cfg2", dict(D=128, N=1536, Hq=1, Hkv=1, Cq=1, Ck=57, r=17, block=512, kmeans_iters=1)),
    "lists_two_blocks": ("cfg2", dict(N=512, Hq=2, Hkv=1, Cq=3, Ck=17, r=4, block=256, kmeans_iters=1)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_chain_lists(name, monkeypatch):
    monkeypatch.setitem(base.CASES, name, CASES[name])
    base.run_case(name, with_bwd=True)


def test_backward_twice_on_one_state():
    w = small("cfg2", N=1024, Hq=2, Hkv=1, Cq=8, Ck=32, r=3, block=128, kmeans_iters=1)
    d = generate(w, need_dO=True)
    p = dataclasses.replace(mb.params_for(w), flags=mb.FLAG_KEEP_FWD_STATE)
    qc, aq, ak = (torch.tensor(x).cuda() for x in base.oracle_clustering(w, d, p))
    Q, K, V, dO = (base.dev(d[x], p) for x in ("Q", "K", "V", "dO"))
    ws = torch.empty(mb.muse_workspace_bytes(p, mb.WS_BWD)[1], dtype=torch.uint8, device="cuda")

    def backward(p, fwd, ws):
        O, LSE, selc, selb = fwd
        return mb.muse_bwd(p, Q, K, V, O, LSE, dO, qc, aq, ak, selc, selb, ws=ws)

    fwd = mb.muse_fwd(p, Q, K, V, qc, aq, ak, ws=ws)
    grads = [backward(p, fwd, ws) for _ in range(3)]
    # and without a state
    grads.append(backward(dataclasses.replace(p, flags=0), fwd, torch.empty_like(ws)))
    for got in grads[1:]:
        assert all(torch.equal(a, b) for a, b in zip(got, grads[0]))


def test_forward_and_backward_again_in_one_workspace():
    w = small("cfg2", N=1024, Hq=2, Hkv=1, Cq=8, Ck=32, r=3, block=128, kmeans_iters=1)
    d = generate(w, need_dO=True)
    p = dataclasses.replace(mb.params_for(w), flags=mb.FLAG_KEEP_FWD_STATE)
    qc, aq, ak = (torch.tensor(x).cuda() for x in base.oracle_clustering(w, d, p))
    Q, K, V, dO = (base.dev(d[x], p) for x in ("Q", "K", "V", "dO"))
    ws = torch.empty(mb.muse_workspace_bytes(p, mb.WS_BWD)[1], dtype=torch.uint8, device="cuda")
    grads = []
    for _ in range(2):
        O, LSE, selc, selb = mb.muse_fwd(p, Q, K, V, qc, aq, ak, ws=ws)
        grads.append(mb.muse_bwd(p, Q, K, V, O, LSE, dO, qc, aq, ak, selc, selb, ws=ws))
    for a, b in zip(*grads):
        assert torch.equal(a, b)
