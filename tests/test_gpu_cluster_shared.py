"""Clustering with queries and keys in the same launches (small problems) against each side alone, bit for bit: sides of different numbers
of heads and clusters, odd lengths, both types and head dimensions, one iteration and none.  And the launches that clear and cast
several arrays, whose ends fall inside 16 bytes."""
import pytest
import torch

from paper_2509_10406_amd import binding as mb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("B,Hq,Hkv,N,D,Cq,Ck,iters", [
    (1, 1, 1, 1024, 64, 3, 70, 3), (1, 4, 1, 1496, 64, 33, 5, 2), (2, 2, 1, 520, 128, 4, 9, 3), (1, 3, 3, 1000, 128, 1, 16, 1), (1, 2, 2, 264, 64, 7, 7, 0)])
def test_shared_launches(dtype, B, Hq, Hkv, N, D, Cq, Ck, iters):
    g = torch.Generator(device="cuda").manual_seed(1)
    p = mb.Params(B=B, Hq=Hq, Hkv=Hkv, N=N, D=D, Cq=Cq, Ck=Ck, r=1, k2=1, kmeans_iters=iters, dtype=mb.FP32 if dtype == "fp32" else mb.BF16,
                  grad_dtype=mb.FP32)
    Q, K = (torch.randn(B, H, N, D, generator=g, device="cuda").to(p.torch_dtype) for H in (Hq, Hkv))
    pick = lambda H, C: torch.rand(B, H, N, generator=g, device="cuda").argsort(-1)[..., :C].to(torch.int32).contiguous()
    qi, ki = pick(Hq, Cq), pick(Hkv, Ck)
    qc, qa, kc, ka = mb.muse_cluster(p, Q, K, qi, ki)
    qc1, qa1, _, _ = mb.muse_cluster(p, Q, None, qi, None)
    _, _, kc1, ka1 = mb.muse_cluster(p, None, K, None, ki)
    assert torch.equal(qc, qc1) and torch.equal(qa, qa1) and torch.equal(kc, kc1) and torch.equal(ka, ka1)
    assert int(qa.min()) >= 0 and int(qa.max()) < Cq and int(ka.min()) >= 0 and int(ka.max()) < Ck


@pytest.mark.parametrize("shared,dtype,Hq,Hkv,N,Cq,Ck", [
    (True, mb.BF16, 2, 2, 2048, 8, 16), (True, mb.FP32, 1, 1, 2048, 16, 32),
    # more than a round of workgroups together, a long update beside a long assignment: 30 to 44 % slower in shared launches
    (False, mb.BF16, 56, 14, 1824, 7, 32), (False, mb.BF16, 24, 6, 15064, 9, 2), (False, mb.FP32, 3, 3, 3248, 2, 105),
    (False, mb.BF16, 16, 16, 4096, 16, 64)])  # too many pairs
def test_which_problems_share(shared, dtype, Hq, Hkv, N, Cq, Ck):
    g = torch.Generator(device="cuda").manual_seed(4)
    p = mb.Params(B=1, Hq=Hq, Hkv=Hkv, N=N, D=64, Cq=Cq, Ck=Ck, r=1, k2=1, kmeans_iters=10, dtype=dtype)
    Q, K = (torch.randn(1, H, N, 64, generator=g, device="cuda").to(p.torch_dtype) for H in (Hq, Hkv))
    qi, ki = (torch.rand(1, H, N, generator=g, device="cuda").argsort(-1)[..., :C].to(torch.int32).contiguous() for H, C in ((Hq, Cq), (Hkv, Ck)))
    mb.muse_profile_enable(True)
    try:
        out = mb.muse_cluster(p, Q, K, qi, ki)
        launches = mb.muse_profile_report()["k_assign_bf16" if dtype == mb.BF16 else "k_assign_f32"][0]
    finally:
        mb.muse_profile_enable(False)
    assert launches == (11 if shared else 22)
    assert all(torch.equal(a, b) for a, b in zip(out, mb.muse_cluster(p, Q, K, qi, ki)))
    one = mb.muse_cluster(p, Q, None, qi, None)[:2] + mb.muse_cluster(p, None, K, None, ki)[2:]
    assert all(torch.equal(a, b) for a, b in zip(out, one))


@pytest.mark.parametrize("offset", [0, 1, 2])
def test_outputs_at_any_word(offset):
    """Selections and bf16 gradients that begin between 16-byte boundaries, and end between them, surrounded by words that stay."""
    p = mb.Params(B=1, Hq=1, Hkv=1, N=264, D=64, Cq=2, Ck=3, r=3, k2=1, block=33, kmeans_iters=1, dtype=mb.BF16, grad_dtype=mb.BF16)
    g = torch.Generator(device="cuda").manual_seed(2)
    Q, K, V, dO = (torch.randn(1, 1, 264, 64, generator=g, device="cuda").bfloat16() for _ in range(4))
    qc, qa, kc, ka = mb.muse_cluster(p, Q, K, torch.tensor([[[0, 100]]], dtype=torch.int32, device="cuda"),
                                     torch.tensor([[[0, 90, 200]]], dtype=torch.int32, device="cuda"))
    want = mb.muse_fwd(p, Q, K, V, qc, qa, ka)
    grads = mb.muse_bwd(p, Q, K, V, want[0], want[1], dO, qc, qa, ka, want[2], want[3])
    bufs = [torch.full((264 * 3 + 16,), 77, dtype=torch.int32, device="cuda") for _ in range(2)]
    selc, selb = (b[4 + offset : 4 + offset + 264 * 3].view(1, 1, 264, 3) for b in bufs)
    got = mb.muse_fwd(p, Q, K, V, qc, qa, ka, out=(torch.empty_like(want[0]), torch.empty_like(want[1]), selc, selb.view(1, 1, 264, 3, 1)))
    assert torch.equal(got[2], want[2]) and torch.equal(got[3], want[3]) and torch.equal(got[0], want[0])
    for b in bufs:
        assert (b[: 4 + offset] == 77).all() and (b[4 + offset + 264 * 3 :] == 77).all()
    gb = [torch.full((264 * 64 + 16,), 5.0, dtype=torch.bfloat16, device="cuda") for _ in range(3)]
    outs = [b[4 + offset : 4 + offset + 264 * 64].view(1, 1, 264, 64) for b in gb]
    mb.muse_bwd(p, Q, K, V, want[0], want[1], dO, qc, qa, ka, want[2], want[3], out=tuple(outs))
    for b, o, w in zip(gb, outs, grads):
        assert torch.equal(o, w) and (b[: 4 + offset] == 5).all() and (b[4 + offset + 264 * 64 :] == 5).all()
