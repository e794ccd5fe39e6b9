"""The backward on two streams, whose last far-field kernels add to gradients that the other stream makes: the bits of the backward on one
stream, with dK and dV of the block diagonal first (no retrieval, or blocks that are long for the far field) and with dQ first, with
and without kept state, in one chunk of heads and in several."""
import pytest
import torch

from paper_2509_10406_amd import binding as mb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [mb.BF16, mb.FP32])
@pytest.mark.parametrize("D,N,block,C,r,flags,chunks", [
    (64, 4096, 2048, 16, 0, mb.FLAG_KEEP_FWD_STATE, False),
    (64, 4096, 2048, 16, 2, mb.FLAG_KEEP_FWD_STATE, False),
    (128, 2048, 1024, 24, 1, 0, False),
    (64, 2048, 256, 64, 8, mb.FLAG_KEEP_FWD_STATE, False),
    (128, 1024, 64, 40, 4, 0, False),
    (64, 2048, 1024, 16, 2, 0, True),
    (64, 2048, 256, 16, 0, 0, True),
])
def test_streams(dtype, D, N, block, C, r, flags, chunks):
    g = torch.Generator(device="cuda").manual_seed(3)
    p = mb.Params(B=1, Hq=4, Hkv=2, N=N, D=D, Cq=C, Ck=C, r=r, k2=1, block=block, kmeans_iters=1, dtype=dtype, grad_dtype=dtype, flags=flags)
    Q, K, V, dO = (torch.randn(1, h, N, D, generator=g, device="cuda").to(p.torch_dtype) for h in (4, 2, 2, 4))
    init = [torch.stack([torch.randperm(N, generator=g, device="cuda")[:C] for _ in range(h)]).int().view(1, h, C) for h in (4, 2)]
    qc, aq, _, ak = mb.muse_cluster(p, Q, K, *init)
    ws = torch.empty(mb.muse_workspace_bytes(p, mb.WS_BWD)[0 if chunks else 1], dtype=torch.uint8, device="cuda")

    def both():
        O, LSE, selc, selb = mb.muse_fwd(p, Q, K, V, qc, aq, ak, ws=ws if flags else None)
        return [x.clone() for x in mb.muse_bwd(p, Q, K, V, O, LSE, dO, qc, aq, ak, selc, selb, ws=ws)]

    mb.muse_profile_enable(True)  # one stream
    try:
        want = both()
    finally:
        mb.muse_profile_enable(False)
    for _ in range(5):
        assert all(torch.equal(a, b) for a, b in zip(both(), want))
