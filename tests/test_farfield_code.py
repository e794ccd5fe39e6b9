"""The machine code of the far field's kernels that load to LDS by hand, compiled here for gfx950 with the library's flags: what these
loads rely on and the compiler does not check.
  - m0 carries their address and nothing else uses it; the base is not in registers that the vector pipe wrote within five wait states
  - no scalar register is spilled (it would come back through the vector pipe), and no vector register either, up to the forms of
    k_farfield_tiles that are listed here with the number that they spill: a reload makes the wave wait for the tiles on their way
  - k_farfield_tiles waits for its tiles by count: what a wait leaves on its way are whole tiles, and what it waits for is a whole one"""
import re
import subprocess

import pytest

from paper_2509_10406_amd import build
from tests.test_attn_bwd_code import faults, functions

# vector registers spilled by k_farfield_tiles: (head dim, list, tiles per wave)
SPILLED = {(64, 8, 6): 6, (64, 16, 6): 5, (64, 32, 6): 17, (64, 8, 8): 6, (64, 16, 8): 4, (64, 32, 8): 7,
           (128, 32, 6): 2, (128, 8, 8): 4, (128, 16, 8): 5, (128, 32, 8): 2}


def code_of(source, tmp_path):
    out = str(tmp_path / "code.s")
    subprocess.run(["hipcc", *build.FLAGS, "--offload-device-only", "-S", f"{build.CSRC}/{source}", "-o", out], check=True, stderr=subprocess.DEVNULL)
    return open(out).read()


def form(name):
    """The numbers among a kernel's template arguments."""
    return tuple(int(x) for x in re.findall(r"Li(\d+)E", name))


def counted(ins, pred, D):
    """The counted waits of a kernel, and those that do not leave whole tiles on their way or do not wait for a whole one: a tile of scores
    is two planes of D / 16 loads of 16 bytes and, behind them, one of 4 bytes; a tile of values is D / 16 loads of 16 bytes."""
    rows, waits, wrong = D // 16, 0, []

    def tile(loads, at):  # the loads of the tile whose last load is loads[at] (0: no whole tile), the list running backwards
        scores = loads[at:at + 1] == (False,)
        run = loads[at + scores:][:2 * rows if scores else rows]
        return scores + len(run) if len(run) == (2 * rows if scores else rows) and all(run) else 0

    for k, x in enumerate(ins):
        m = x.asm and x.op == "s_waitcnt" and re.fullmatch(r"vmcnt\((\d+)\)", x.args)
        left = int(m[1]) if m else 0
        if not left:
            continue
        waits += 1
        todo, seen = [(p, ()) for p in pred[k]], set()
        while todo:  # the loads in front of the wait on every path, last one first; whether they are of 16 bytes
            at, loads = todo.pop()
            if (at, loads) in seen:
                continue
            seen.add((at, loads))
            if ins[at].asm and ins[at].op.startswith("global_load_lds_dword"):
                loads += (ins[at].op.endswith("x4"),)
            if pred[at] and len(loads) <= left + 2 * rows:
                todo += [(p, loads) for p in pred[at]]
                continue
            done = 0
            while done < left and (n := tile(loads, done)):
                done += n
            if done != left or not tile(loads, done):
                wrong.append(f"{k}: vmcnt({left}) behind {loads}")
    return waits, wrong


@pytest.mark.parametrize("source, kernel, count", [
    ("farfield_tiles.hip", "k_farfield_tiles", 30),  # head dims x lists of 8, 16, 32 x tiles per wave
    ("chain_grads.hip", "k_chain_gradsI", 8),        # head dims x chains per wave x waves
])
def test_loads_to_lds(source, kernel, count, tmp_path):
    code = code_of(source, tmp_path)
    got = {name: f for name, f in functions(code).items() if kernel in name}
    assert len(got) == count
    for name, (ins, pred) in got.items():
        assert any(x.op == "global_load_lds_dwordx4" for x in ins), name
        assert not (f := faults(ins, pred)), (name, f[:5])
        waits, wrong = counted(ins, pred, form(name)[0])
        assert not wrong, (name, wrong[:3])
        # tiles of one wave but the last are waited for by count
        assert waits == 0 if kernel != "k_farfield_tiles" else waits >= form(name)[2] - 1, (name, waits)
    spilled = {m[1]: m[2:] for m in re.findall(r"(\.name:\s+(\S*)[\s\S]*?\.sgpr_spill_count:\s+(\d+)[\s\S]*?\.vgpr_spill_count:\s+(\d+))", code)}
    kept = {name: s for name, s in spilled.items() if kernel in name and not name.endswith(".kd")}
    assert len(kept) == count
    for name, (sgprs, vgprs) in kept.items():
        most = SPILLED.get(form(name)[:3], 0) if kernel == "k_farfield_tiles" else 0
        assert sgprs == "0" and int(vgprs) <= most, (name, sgprs, vgprs)


ASM = "\t;;#ASMSTART\n%s\t;;#ASMEND\n"
ROWS, WORDS = (ASM % f"\ts_mov_b32 m0, s5\n\ts_nop 0\n\tglobal_load_lds_{what} v2, s[38:39]\n" for what in ("dwordx4", "dword"))
SCORES, VALUES = 8 * ROWS + WORDS, 4 * ROWS


@pytest.mark.parametrize("body, left, wrong", [
    (SCORES + SCORES, 9, False),
    (SCORES + SCORES, 8, True),
    (SCORES + SCORES, 10, True),
    (SCORES + VALUES + VALUES, 8, False),
    (SCORES + VALUES + VALUES, 4, False),
    (SCORES + VALUES + VALUES, 9, True),
    (SCORES + VALUES, 5, True),
    (VALUES, 4, True),  # nothing is waited for
    (SCORES + VALUES + "\ts_cbranch_scc1 .LBB0_1\n" + VALUES + ".LBB0_1:\n", 8, True),  # one tile of values too few on one path
])
def test_the_check_sees_what_it_is_for(body, left, wrong):
    ins, pred = functions("_Zk:\n" + body + ASM % f"\ts_waitcnt vmcnt({left})\n" + "\ts_endpgm\n.Lfunc_end0:\n")["_Zk"]
    waits, got = counted(ins, pred, 64)
    assert waits == 1 and bool(got) == wrong, got
