"""GPU parity of the bf16 backward where the gradients of the accumulated cells (cell_grads.hip) change their path: groups
of one and of several stages of 32 queries, units of 16 clusters that are not full, one to ten units (test_gpu_cell_walk.py: the two ways
the key blocks are taken).  Tolerances are those of the parity suite."""
import pytest

import tests.test_gpu_muse as base

pytestmark = pytest.mark.gpu

CASES = {
    # one query cluster: groups of a whole block of 256 queries, eight stages; 17 clusters: a unit with one
    "cells_passes": ("cfg2", dict(N=1024, Hq=2, Hkv=1, Cq=1, Ck=17, r=2, block=256, kmeans_iters=1)),
    # groups of some 32 queries, one or two stages; 150 clusters, ten units
    "cells_units": ("cfg2", dict(N=1024, Hq=2, Hkv=2, Cq=4, Ck=150, r=4, block=128, kmeans_iters=1)),
    "cells_d128_passes": ("cfg2", dict(D=128, N=1024, Hq=2, Hkv=1, Cq=1, Ck=33, r=2, block=256, kmeans_iters=1)),
    "cells_d128_r0": ("cfg2", dict(D=128, N=768, Hq=1, Hkv=1, Cq=6, Ck=15, r=0, block=96, kmeans_iters=1)),
}
base.REACH.update({"cells_passes": dict(group=193), "cells_d128_passes": dict(group=193)})


@pytest.mark.parametrize("name", list(CASES))
def test_cell_gradients(name, monkeypatch):
    monkeypatch.setitem(base.CASES, name, CASES[name])
    base.run_case(name, with_bwd=True)
