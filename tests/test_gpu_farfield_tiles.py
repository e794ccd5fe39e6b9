"""GPU parity of the far-field forward of bf16 inputs (k_farfield_tiles) where its tiles of 32 key clusters end: one cluster, one
less and one more than a tile, three tiles with one cluster in the last, at both head dimensions and at every list length (8, 16
and 32 candidates).  Tolerances are those of the parity suite."""
import pytest

import tests.test_gpu_muse as base

pytestmark = pytest.mark.gpu

CASES = {f"ff_d{D}_ck{Ck}_r{r}": ("cfg2", dict(D=D, N=1024, Hq=2, Hkv=1, Cq=3, Ck=Ck, r=r, block=128, kmeans_iters=1))
         for D in (64, 128) for Ck, r in ((1, 1), (31, 3), (32, 16), (33, 8), (65, 17))}


@pytest.mark.parametrize("name", list(CASES))
def test_far_field_tiles(name, monkeypatch):
    monkeypatch.setitem(base.CASES, name, CASES[name])
    base.run_case(name, with_bwd=False)
