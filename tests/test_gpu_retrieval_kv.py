"""GPU parity of the bf16 retrieval where its kernels change form.  Query side (retrieval_q.hip): 64 keys staged at a time,
so pairs of up to 64 keys and of several stages.  Key/value gradients (retrieval_kv.hip): pairs of up to
32 keys (the waves share the hits), 33 to 64 (a wave per key tile) and more (several key groups), several hit slices, one
hit, and grouped queries; D = 128 with later slices; and the longer slices that calls of many hits have.  Tolerance: the
parity suite's; at D = 128, where dQ comes near it, the oracle's bound on the rounding of its bf16 operands."""
import numpy as np
import pytest
import torch

import tests.test_gpu_muse as base
from paper_2509_10406_amd import binding as mb
from paper_2509_10406_amd.inputs import generate, small

pytestmark = pytest.mark.gpu

CASES = {
    "kv_pairs40_gqa": ("cfg2", dict(N=2048, Hq=4, Hkv=2, Cq=4, Ck=6, r=3, k2=2, block=256, kmeans_iters=1)),
    "kv_pairs250": ("cfg2", dict(N=4096, Hq=2, Hkv=1, Cq=3, Ck=2, r=1, block=512, kmeans_iters=1)),
    "kv_single_hits": ("cfg2", dict(N=512, Hq=1, Hkv=1, Cq=8, Ck=60, r=1, block=64, kmeans_iters=1)),
}
OWN_OUTPUTS = {
    "kv_d128_pairs250": ("cfg5", dict(N=4096, Hq=2, Hkv=1, Cq=3, Ck=2, r=1, block=512, kmeans_iters=1)),
    "kv_d128_pairs85": ("cfg5", dict(N=4096, Hq=2, Hkv=1, Cq=6, Ck=6, r=2, block=512, kmeans_iters=1)),
}
base.REACH.update({"kv_pairs40_gqa": dict(pair_keys=33, pair_hits=512), "kv_pairs250": dict(pair_keys=129, pair_hits=512),
                   # a second slice from 8 tiles of 32 hits on
                   "kv_d128_pairs250": dict(pair_keys=129, pair_hits=1024), "kv_d128_pairs85": dict(pair_keys=65, pair_hits=256)})


@pytest.mark.parametrize("name", list(CASES))
def test_retrieval_key_value_gradients(name, monkeypatch):
    monkeypatch.setitem(base.CASES, name, CASES[name])
    base.run_case(name, with_bwd=True)


@pytest.mark.parametrize("name", list(OWN_OUTPUTS))
def test_retrieval_key_value_gradients_d128(name, monkeypatch):
    monkeypatch.setitem(base.CASES, name, OWN_OUTPUTS[name])
    base.run_case(name, with_bwd=True, own_outputs=True)


@pytest.mark.parametrize("kw,tiles", [(dict(Hq=32, Hkv=8, N=4096, Ck=16, r=16), 16), (dict(Hq=16, Hkv=4, N=3072, Ck=20, r=16), 6),
                                      (dict(Hq=16, Hkv=4, N=4096, D=128, Ck=16, r=16), 8)])
def test_long_slices(kw, tiles):
    """A call of many hits cuts a pair's hits into slices of up to 16 tiles of 32; one KV group of it, run alone, into slices
    of four.  Both must give the group the same dK and dV, up to the rounding of the cell gradients, which are stored in
    bf16 (2^-8 at most, 2^-9 of the norm) and summed in an order of their own in either call."""
    w = small("cfg2", Cq=8, block=kw["N"] // 8, kmeans_iters=1, **kw)
    d = generate(w, need_dO=True)
    assert w.Hq * w.N * w.r // (32 * 4096) == tiles
    G, g = w.Hq // w.Hkv, 2

    def run(hq, hk):
        p = mb.Params(B=1, Hq=hq.stop - hq.start, Hkv=hk.stop - hk.start, N=w.N, D=w.D, Cq=w.Cq, Ck=w.Ck, r=w.r, block=w.Bs, kmeans_iters=1)
        Q, dO = (d[x][:, hq].bfloat16().cuda().contiguous() for x in ("Q", "dO"))
        K, V = (d[x][:, hk].bfloat16().cuda().contiguous() for x in ("K", "V"))
        qc, qa, _, ka = mb.muse_cluster(p, Q, K, d["q_init_idx"][:, hq].cuda().contiguous(), d["k_init_idx"][:, hk].cuda().contiguous())
        O, LSE, selc, selb = mb.muse_fwd(p, Q, K, V, qc, qa, ka)
        return (O, selc, selb, *mb.muse_bwd(p, Q, K, V, O, LSE, dO, qc, qa, ka, selc, selb))

    every, alone = run(slice(0, w.Hq), slice(0, w.Hkv)), run(slice(g * G, (g + 1) * G), slice(g, g + 1))
    assert torch.equal(every[0][:, g * G:(g + 1) * G], alone[0]) and torch.equal(every[2][:, g * G:(g + 1) * G], alone[2])
    sc, sb = (x.cpu().numpy().reshape(-1) for x in alone[1:3])
    ok = sb >= 0
    assert np.bincount(sb[ok] * w.Ck + sc[ok]).max() >= 2 * 32 * tiles, "no pair has a second slice"
    for i, what in ((4, "dK"), (5, "dV")):
        a, b = every[i][:, g].double(), alone[i][:, 0].double()
        err = ((a - b).norm() / b.norm()).item()
        print(f"{what}: {err:.1e}")
        assert err <= 2 * 2.0 ** -9, (what, err)
