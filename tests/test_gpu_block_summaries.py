"""GPU parity of the per-block summaries of retrieved chains (k_block_summaries_mx, bf16 inputs) where a cell's keys change their path:
cells of up to one, two and three chunks of 8 keys, longer ones, empty ones, at both head dimensions and both register budgets, with
more than 32 chains per key cluster.  They are seen through component 2 of the forward and both its backwards.  Tolerances are those
of the parity suite."""
import pytest

import tests.test_gpu_muse as base

pytestmark = pytest.mark.gpu

# Ck key clusters in blocks of `block` keys: cells of block / Ck keys on average, from 0 to several times that
CASES = {f"cells_d{D}_{block // Ck}": ("cfg2", dict(D=D, N=4 * block, Hq=2, Hkv=1, Cq=40, Ck=Ck, r=4, block=block, kmeans_iters=1))
         for D in (64, 128) for block, Ck in ((256, 64), (480, 40), (480, 24), (512, 10))}


@pytest.mark.parametrize("name", list(CASES))
def test_cells(name, monkeypatch):
    monkeypatch.setitem(base.CASES, name, CASES[name])
    base.run_case(name, with_bwd=True)
