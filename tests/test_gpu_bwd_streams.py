"""The backward on two streams, where far-field gradients meet the block diagonal's that the other stream makes: the bits of the backward on
one stream, with the keys' and values' scattered behind both streams and (many rows and waves) added by the kernel that makes them, with
and without retrieval and kept state, in one chunk of heads and in several."""
import pytest
import torch

from paper_2509_10406_amd import binding as mb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [mb.BF16, mb.FP32])
@pytest.mark.parametrize("D,N,block,C,r,flags,chunks,H", [
    (64, 4096, 2048, 16, 0, mb.FLAG_KEEP_FWD_STATE, False, 2),
    (64, 4096, 2048, 16, 2, mb.FLAG_KEEP_FWD_STATE, False, 2),
    (128, 2048, 1024, 24, 1, 0, False, 2),
    (64, 2048, 256, 64, 8, mb.FLAG_KEEP_FWD_STATE, False, 2),
    (128, 1024, 64, 40, 4, 0, False, 2),
    (64, 2048, 1024, 16, 2, 0, True, 2),
    (64, 2048, 256, 16, 0, 0, True, 2),
    (64, 8192, 1024, 32, 2, mb.FLAG_KEEP_FWD_STATE, False, 32),  # added: 7168 waves, 117 MB of rows
    (128, 4096, 512, 24, 0, 0, False, 32),
])
def test_streams(dtype, D, N, block, C, r, flags, chunks, H):
    g = torch.Generator(device="cuda").manual_seed(3)
    p = mb.Params(B=1, Hq=2 * H if H < 32 else H, Hkv=H, N=N, D=D, Cq=C, Ck=C, r=r, k2=1, block=block, kmeans_iters=1, dtype=dtype, grad_dtype=dtype, flags=flags)
    Q, K, V, dO = (torch.randn(1, h, N, D, generator=g, device="cuda").to(p.torch_dtype) for h in (p.Hq, H, H, p.Hq))
    init = [torch.stack([torch.randperm(N, generator=g, device="cuda")[:C] for _ in range(h)]).int().view(1, h, C) for h in (p.Hq, H)]
    qc, aq, _, ak = mb.muse_cluster(p, Q, K, *init)
    ws = torch.empty(mb.muse_workspace_bytes(p, mb.WS_BWD)[0 if chunks else 1], dtype=torch.uint8, device="cuda")

    def both():
        O, LSE, selc, selb = mb.muse_fwd(p, Q, K, V, qc, aq, ak, ws=ws if flags else None)
        return [x.clone() for x in mb.muse_bwd(p, Q, K, V, O, LSE, dO, qc, aq, ak, selc, selb, ws=ws)]

    mb.muse_profile_enable(True)  # one stream
    try:
        want = both()
        assert ("k_scatter_rows" in mb.muse_profile_report()) == (H == 2 or dtype == mb.FP32)
    finally:
        mb.muse_profile_enable(False)
    for _ in range(5):
        assert all(torch.equal(a, b) for a, b in zip(both(), want))
