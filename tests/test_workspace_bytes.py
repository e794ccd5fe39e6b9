"""CPU-only: what fp32 calls need of a workspace.  The sizes are those of a layout without an inverse index and without
shared pairs (a bit per (query, key block, key cluster) instead): programs have reserved them, so they are an upper bound."""
import pytest

from paper_2509_10406_amd import binding as mb

SHAPES = [  # kw, (least, preferred) bytes of the forward, of the backward
    (dict(Hq=1, Hkv=1, N=2048, D=64, Cq=16, Ck=32, r=2), (6657536, 6657536), (11965952, 11965952)),
    (dict(Hq=4, Hkv=4, N=8192, D=64, Cq=32, Ck=128, r=4), (96933632, 188850944), (152884992, 333570816)),
    (dict(Hq=16, Hkv=16, N=65536, D=64, Cq=256, Ck=1024, r=8), (6079457792, 35492997632), (8950983168, 66770446848)),
    (dict(Hq=16, Hkv=16, N=65536, D=64, Cq=128, Ck=128, r=8), (3442895360, 5721643520), (4421347840, 8475466240)),
    (dict(Hq=16, Hkv=4, N=65536, D=64, Cq=256, Ck=1024, r=8), (11551817216, 35082649088), (19701874176, 65957445120)),
    (dict(Hq=16, Hkv=16, N=65536, D=128, Cq=256, Ck=1024, r=8), (10911296000, 68510558720), (16467700224, 130658609664)),
    (dict(Hq=16, Hkv=16, N=65536, D=64, Cq=256, Ck=1024, r=0), (4022872576, 33436412416), (6865037824, 64684501504)),
]


@pytest.mark.parametrize("kw,fwd,bwd", SHAPES)
def test_fp32_workspace_stays_within(kw, fwd, bwd):
    p = mb.Params(B=1, dtype=mb.FP32, grad_dtype=mb.FP32, **kw)
    for which, most in ((mb.WS_FWD, fwd), (mb.WS_BWD, bwd)):
        least, preferred = mb.muse_workspace_bytes(p, which)
        assert least <= most[0] and preferred <= most[1], (which, least, preferred)
