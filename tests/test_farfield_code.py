"""The machine code of the far field's kernels that load to LDS by hand, compiled here for gfx950 with the library's flags: what these
loads rely on and the compiler does not check (m0 carries their address and nothing else uses it; the base is not in registers
that the vector pipe wrote within five wait states), and that no kernel with such loads spills a scalar register, which would
come back through the vector pipe, or, where what it brings is waited for in groups, a vector register."""
import re
import subprocess

import pytest

from paper_2509_10406_amd import build
from tests.test_attn_bwd_code import faults, functions


@pytest.mark.parametrize("source, kernel, count, spills", [
    ("farfield_tiles.hip", "k_farfield_tiles", 30, True),  # head dims x lists of 8, 16, 32 x tiles per wave
    ("chain_grads.hip", "k_chain_gradsI", 8, False),       # head dims x chains per wave x waves
])
def test_loads_to_lds(source, kernel, count, spills, tmp_path):
    out = str(tmp_path / "code.s")
    subprocess.run(["hipcc", *build.FLAGS, "--offload-device-only", "-S", f"{build.CSRC}/{source}", "-o", out], check=True, stderr=subprocess.DEVNULL)
    code = open(out).read()
    got = {name: f for name, f in functions(code).items() if kernel in name}
    assert len(got) == count
    for name, (ins, pred) in got.items():
        assert any(x.op == "global_load_lds_dwordx4" for x in ins), name
        assert not (f := faults(ins, pred)), (name, f[:5])
    spilled = {m[1]: m[2:] for m in re.findall(r"(\.name:\s+(\S*)[\s\S]*?\.sgpr_spill_count:\s+(\d+)[\s\S]*?\.vgpr_spill_count:\s+(\d+))", code)}
    kept = {name: s for name, s in spilled.items() if kernel in name and not name.endswith(".kd")}
    assert len(kept) == count and all(s[0] == "0" and (spills or s[1] == "0") for s in kept.values()), kept
