"""GPU parity of the bf16 cell gradients where the walk over the key blocks (cell_grads.hip) changes its path: empty groups
(stages of no rows, first and last among them), groups of exactly one and of several stages of 32 queries, sixteen key
blocks, a second workgroup of units with one unit in it.  Tolerances are those of the parity suite."""
import pytest

import tests.test_gpu_muse as base

pytestmark = pytest.mark.gpu

CASES = {
    "walk_empty_groups": ("cfg2", dict(N=512, Hq=2, Hkv=1, Cq=24, Ck=65, r=2, block=32, kmeans_iters=1)),
    "walk_one_stage": ("cfg2", dict(N=256, Hq=1, Hkv=1, Cq=1, Ck=16, r=1, block=32, kmeans_iters=1)),
    "walk_d128": ("cfg2", dict(D=128, N=768, Hq=2, Hkv=2, Cq=9, Ck=130, r=4, block=64, kmeans_iters=1)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_cell_walk(name, monkeypatch):
    monkeypatch.setitem(base.CASES, name, CASES[name])
    base.run_case(name, with_bwd=True)
