"""GPU parity of the bf16 cell gradients where the accumulation over the key blocks (cell_grads.hip) changes its path.  The waves of a
workgroup take a key block each where there are few units of 16 key clusters ("apart"), else each walks the key blocks of a unit of
its own ("walk"); for both: empty groups (stages of no rows, first and last among them), groups of exactly one and of several stages of
32 queries, sixteen key blocks (two rounds of eight) and a few, units that are not full, workgroups that are not.  Tolerances are those
of the parity suite."""
import pytest

import tests.test_gpu_muse as base
from paper_2509_10406_amd.inputs import small

pytestmark = pytest.mark.gpu

CASES = {
    "walk_empty_groups": ("apart", "cfg2", dict(N=512, Hq=2, Hkv=1, Cq=24, Ck=65, r=2, block=32, kmeans_iters=1)),
    "walk_one_stage": ("apart", "cfg2", dict(N=256, Hq=1, Hkv=1, Cq=1, Ck=16, r=1, block=32, kmeans_iters=1)),
    "walk_d128": ("apart", "cfg2", dict(D=128, N=768, Hq=2, Hkv=2, Cq=9, Ck=130, r=4, block=64, kmeans_iters=1)),
    "apart_stages": ("apart", "cfg2", dict(N=1440, Hq=2, Hkv=1, Cq=1, Ck=20, r=2, block=480, kmeans_iters=1)),
    "apart_d128_stages": ("apart", "cfg2", dict(D=128, N=1536, Hq=2, Hkv=1, Cq=2, Ck=20, r=2, block=256, kmeans_iters=1)),
    "walk_nb16": ("walk", "cfg2", dict(N=512, Hq=2, Hkv=1, Cq=33, Ck=130, r=2, block=32, kmeans_iters=1)),
    "walk_units": ("walk", "cfg2", dict(N=1024, Hq=4, Hkv=2, Cq=33, Ck=130, r=4, block=128, kmeans_iters=1)),
    "walk_stages": ("walk", "cfg2", dict(N=4096, Hq=4, Hkv=2, Cq=4, Ck=1030, r=4, block=512, kmeans_iters=1)),
    "walk_two_blocks": ("walk", "cfg2", dict(N=512, Hq=2, Hkv=1, Cq=2, Ck=40, r=2, block=256, kmeans_iters=1)),
    "walk_d128_units": ("walk", "cfg2", dict(D=128, N=768, Hq=4, Hkv=2, Cq=33, Ck=130, r=3, block=96, kmeans_iters=1)),
    "walk_d128_stages": ("walk", "cfg2", dict(D=128, N=2048, Hq=4, Hkv=2, Cq=4, Ck=1030, r=4, block=256, kmeans_iters=1)),
    "walk_d128_three_blocks": ("walk", "cfg2", dict(D=128, N=768, Hq=2, Hkv=1, Cq=3, Ck=50, r=2, block=256, kmeans_iters=1)),
}
base.REACH.update({"apart_stages": dict(group=257), "apart_d128_stages": dict(group=97), "walk_stages": dict(group=97),
                   "walk_d128_stages": dict(group=65), "walk_two_blocks": dict(group=97), "walk_d128_three_blocks": dict(group=65)})


def form(w):
    """The launch's choice (cells_apart)."""
    units, far = w.B * w.Hq * w.Cq * ((w.Ck + 15) // 16), w.N // w.Bs - 1
    return "apart" if far >= (2 if w.D == 64 else 4) and units * ((far + 7) // 8) <= 1024 else "walk"


@pytest.mark.parametrize("name", list(CASES))
def test_cell_walk(name, monkeypatch):
    want_form, cfg, kw = CASES[name]
    assert form(small(cfg, **kw)) == want_form
    monkeypatch.setitem(base.CASES, name, (cfg, kw))
    base.run_case(name, with_bwd=True)
