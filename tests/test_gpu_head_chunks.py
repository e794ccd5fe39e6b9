"""The bits of a call do not depend on the size of its workspace: the smallest one (a KV group at a time), one in between
and the preferred one (all heads at once), at cluster counts where a launch of one head spreads the chains of a word of 32
key clusters over more workgroups than a launch of all heads would need."""
import pytest
import torch

from paper_2509_10406_amd import binding as mb
from paper_2509_10406_amd.inputs import generate, small

pytestmark = pytest.mark.gpu

CASES = {
    "bf16": ("cfg2", dict(N=2048, Hq=8, Hkv=8, Cq=24, Ck=71, r=4, block=256, kmeans_iters=2)),
    "bf16_gqa_k2_2": ("cfg2", dict(N=2048, Hq=8, Hkv=2, Cq=64, Ck=32, r=5, k2=2, block=256, kmeans_iters=2)),
    "bf16_d128_nb12": ("cfg5", dict(N=1536, Hq=4, Hkv=2, Cq=40, Ck=35, r=9, block=128, kmeans_iters=2)),
    # tilt logits: one tile of keys per wave in a chunk of one head, four (two) in a launch of all heads; sizes that end inside both
    "bf16_tilt": ("cfg2", dict(N=16392, Hq=8, Hkv=8, Cq=33, Ck=20, r=1, block=2049, kmeans_iters=1)),
    "bf16_tilt_d128": ("cfg5", dict(N=8200, Hq=8, Hkv=8, Cq=33, Ck=20, r=1, block=1025, kmeans_iters=1)),
    "fp32": ("cfg1", dict(N=1536, Hq=6, Hkv=3, Cq=32, Ck=48, r=3, block=192, kmeans_iters=2)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_bits_do_not_depend_on_the_workspace(name):
    base, kw = CASES[name]
    w = small(base, **kw)
    d = generate(w, need_dO=True)
    p = mb.params_for(w)
    Q, K, V, dO = (d[x].to(p.torch_dtype).cuda().contiguous() for x in ("Q", "K", "V", "dO"))
    qc, qa, _, ka = mb.muse_cluster(p, Q, K, d["q_init_idx"].cuda(), d["k_init_idx"].cuda())
    runs = []
    for share in (1.0, 0.5, 0.0):
        ws = []
        for which in (mb.WS_FWD, mb.WS_BWD):
            mn, pref = mb.muse_workspace_bytes(p, which)
            assert mn < pref
            ws.append(torch.empty(mn + int(share * (pref - mn)), dtype=torch.uint8, device="cuda"))
        O, LSE, selc, selb = mb.muse_fwd(p, Q, K, V, qc, qa, ka, ws=ws[0])
        runs.append((O, LSE, selc, selb, *mb.muse_bwd(p, Q, K, V, O, LSE, dO, qc, qa, ka, selc, selb, ws=ws[1])))
    for other in runs[1:]:
        for what, a, b in zip(("O", "LSE", "selc", "selb", "dQ", "dK", "dV"), runs[0], other):
            assert torch.equal(a, b), f"{what}: {(a.double() - b.double()).abs().max().item():.3e}"
