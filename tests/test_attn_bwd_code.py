"""The machine code of attn_bwd.hip, compiled here for gfx950 with the library's flags: what its hand-written instructions rely on and
the compiler does not check, because it does not look into them.
  - v_mfma with its accumulator in accumulation registers: operands written two wait states earlier by the vector pipe, eleven
    by another matrix instruction; nobody else touches the accumulator until nineteen wait states after the last one
    (the architecture's manually inserted wait states, at the longest figure for any matrix instruction)
  - global_load_lds: m0 carries its LDS address and nothing else in the file uses it; the base is not in registers that the vector
    pipe wrote within five wait states
  - no spilled registers: a spill would put moves in front of the matrix instructions
A wait state is an instruction, s_nop n is n + 1."""
import re
import subprocess

import pytest

from paper_2509_10406_amd import build

REG = re.compile(r"\b([vas])(?:\[(\d+):(\d+)\]|(\d+)\b)|\b(vcc|m0)\b")
READS_M0 = re.compile(r"movrel|gws|s_sendmsg|v_interp|ds_(param|direct)|ds_read_addtid|ds_write_addtid|lds$")


def regs(text):
    out = set()
    for m in REG.finditer(text):
        if m.group(5):
            out.add((m.group(5), 0))
        else:
            a = int(m.group(2) if m.group(4) is None else m.group(4))
            out |= {(m.group(1), n) for n in range(a, int(m.group(3) or a) + 1)}
    return out


class Ins:
    def __init__(self, op, args, asm):
        self.op, self.args, self.asm = op, args, asm
        parts = args.split(", ")
        self.first, self.rest = regs(parts[0]), [regs(p) for p in parts[1:]]
        self.all = self.first.union(*self.rest)
        self.mfma, self.valu = op.startswith("v_mfma"), op.startswith("v_") and not op.startswith(("v_mfma", "v_nop"))
        self.states = int(args.split()[0], 0) + 1 if op == "s_nop" else 1


def functions(text):
    """{name: (instructions, predecessors of each)}"""
    got, name, ins, labels, asm = {}, None, [], {}, False
    for line in text.splitlines():
        if m := re.match(r"(_Z\w+):", line):
            name, ins, labels = m.group(1), [], {}
        elif name is None:
            continue
        elif ";;#ASMSTART" in line or ";;#ASMEND" in line:
            asm = "START" in line
        elif m := re.match(r"(\.LBB\w+):", line):
            labels[m.group(1)] = len(ins)
        elif ".end_amdhsa_kernel" in line or line.startswith(".Lfunc_end"):
            if name not in got:
                pred = [[] for _ in ins]
                for k, (x, target) in enumerate(ins):
                    if target in labels and labels[target] < len(ins):
                        pred[labels[target]].append(k)
                    if x.op not in ("s_branch", "s_endpgm") and k + 1 < len(ins):
                        pred[k + 1].append(k)
                got[name] = ([x for x, _ in ins], pred)
            name = None
        elif m := re.match(r"\s+([a-z][a-z_0-9]+)\b\s*([^;]*)", line):
            ins.append((Ins(m.group(1), m.group(2).strip(), asm), m.group(2).strip() if m.group(1).startswith(("s_cbranch", "s_branch")) else None))
    return got


def before(ins, pred, k, states):
    """The instructions less than `states` wait states in front of k, on every path, with the wait states between."""
    todo, seen = [(p, 0) for p in pred[k]], set()
    while todo:
        at, gap = todo.pop()
        if gap >= states or (at, gap) in seen:
            continue
        seen.add((at, gap))
        yield ins[at], gap
        todo += [(p, gap + ins[at].states) for p in pred[at]]


def faults(ins, pred):
    found = []
    accs = set().union(*(x.first for x in ins if x.mfma and x.asm), set())
    for k, x in enumerate(ins):
        if x.mfma and x.asm:
            operands = x.rest[0] | x.rest[1]
            for y, gap in before(ins, pred, k, 11):
                if (y.valu and gap < 2 or y.mfma) and y.first & operands:
                    found.append(f"{k}: operand of {x.op} written {gap} wait states earlier by {y.op}")
        elif x.all & accs:
            for y, gap in before(ins, pred, k, 19):
                if y.mfma and y.asm and y.first & x.all:
                    found.append(f"{k}: {x.op} {gap} wait states behind the matrix instruction that makes its operand")
        if x.asm and x.op.startswith("global_load_lds"):
            base = {r for r in x.all if r[0] == "s"}
            for y, gap in before(ins, pred, k, 5):
                if y.valu and y.first & base:
                    found.append(f"{k}: base of {x.op} written {gap} wait states earlier by {y.op}")
        elif not (x.asm and x.op == "s_mov_b32") and (("m0", 0) in x.all or READS_M0.search(x.op)):
            found.append(f"{k}: {x.op} uses m0")
    return found


@pytest.fixture(scope="module")
def code(tmp_path_factory):
    src, out = f"{build.CSRC}/attn_bwd.hip", str(tmp_path_factory.mktemp("asm") / "attn_bwd.s")
    subprocess.run(["hipcc", *build.FLAGS, *build.FILE_FLAGS["attn_bwd.hip"], "--offload-device-only", "-S", src, "-o", out], check=True,
                   stderr=subprocess.DEVNULL)
    return open(out).read()


def test_hand_written_instructions(code):
    got = functions(code)
    assert len(got) == 8  # dK / dV at either head dimension and dQ at either, for two types of gradients
    for name, (ins, pred) in got.items():
        assert sum(x.mfma and x.asm for x in ins) >= 24 and any(x.op.startswith("global_load_lds") for x in ins), name
        assert not (f := faults(ins, pred)), (name, f[:5])
    for what in ("sgpr_spill_count", "vgpr_spill_count", "private_segment_fixed_size"):
        assert re.findall(rf"\.{what}:\s+(\d+)", code) == ["0"] * 8, what


MFMA = "\tv_mfma_f32_32x32x16_bf16 a[0:15], v[0:3], v[4:7], a[0:15]\n"
ASM = "\t;;#ASMSTART\n%s\t;;#ASMEND\n"


@pytest.mark.parametrize("body, wrong", [
    ("\tv_cvt_pk_bf16_f32 v4, v9, v10\n\ts_nop 1\n" + ASM % MFMA, 0),
    ("\tv_cvt_pk_bf16_f32 v4, v9, v10\n\ts_nop 0\n" + ASM % MFMA, 1),
    ("\tv_mfma_f32_32x32x16_bf16 v[0:15], v[20:23], v[24:27], 0\n\ts_nop 9\n" + ASM % MFMA, 1),
    (ASM % MFMA + "\ts_nop 15\n\ts_nop 1\n\tv_accvgpr_read_b32 v8, a3\n", 1),
    (ASM % MFMA + "\ts_nop 15\n\ts_nop 2\n\tv_accvgpr_read_b32 v8, a3\n", 0),
    # around a loop: the last instruction of the body stands in front of the first
    (".LBB0_1:\n" + ASM % MFMA + "\ts_nop 3\n\tv_mov_b32_e32 v0, v9\n\ts_cbranch_scc1 .LBB0_1\n", 1),
    (ASM % "\ts_mov_b32 m0, s5\n\ts_nop 0\n\tglobal_load_lds_dwordx4 v2, s[38:39]\n", 0),
    ("\tv_readfirstlane_b32 s38, v3\n" + ASM % "\ts_mov_b32 m0, s5\n\ts_nop 0\n\tglobal_load_lds_dwordx4 v2, s[38:39]\n", 1),
    ("\ts_mov_b32 m0, s3\n\tv_movrels_b32_e32 v1, v2\n", 2),
])
def test_the_check_sees_what_it_is_for(body, wrong):
    ins, pred = functions("_Zk:\n" + body + "\ts_endpgm\n.Lfunc_end0:\n")["_Zk"]
    assert len(faults(ins, pred)) == wrong
