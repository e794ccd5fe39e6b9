"""The machine code of farfield_tiles.hip, compiled here for gfx950 with the library's flags: what its hand-written loads to LDS rely
on and the compiler does not check (m0 carries their address and nothing else uses it; the base is not in registers that
the vector pipe wrote within five wait states), and that no kernel spills a scalar register, which would come back through the vector pipe."""
import re
import subprocess

from paper_2509_10406_amd import build
from tests.test_attn_bwd_code import faults, functions


def test_loads_to_lds(tmp_path):
    out = str(tmp_path / "farfield_tiles.s")
    subprocess.run(["hipcc", *build.FLAGS, "--offload-device-only", "-S", f"{build.CSRC}/farfield_tiles.hip", "-o", out], check=True, stderr=subprocess.DEVNULL)
    code = open(out).read()
    got = functions(code)
    assert len(got) == 30  # head dims x lists of 8, 16, 32 x tiles per wave
    for name, (ins, pred) in got.items():
        assert any(x.op == "global_load_lds_dwordx4" for x in ins) and any(x.op == "global_load_lds_dword" for x in ins), name
        assert not (f := faults(ins, pred)), (name, f[:5])
    assert set(re.findall(r"\.sgpr_spill_count:\s+(\d+)", code)) == {"0"}
