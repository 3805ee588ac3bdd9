"""Wait states around matrix instructions, read from the built library's own device code.

The hardware does not interlock everything: a vector instruction's result may not be an operand of a matrix instruction before
two wait states have passed, and a matrix instruction's result may not be touched by anything but another matrix instruction before
its passes are over.  The compiler inserts the waits for matrix instructions it knows; those written in assembly
(attn_bwd.hip) are opaque to it, and it moves their operands as it likes.  This test follows every path of every kernel."""
import os
import re
import subprocess

import pytest

from paper_2506_23858_amd import build, binding as vb

OBJDUMP = os.path.join(os.path.dirname(os.path.dirname(build.HIPCC)), "llvm", "bin", "llvm-objdump")
OPERAND_WAIT = 2                                          # vector instruction -> operand of a matrix instruction
RESULT_WAIT = {"32x32x16_bf16": 12, "32x32x16_f16": 12, "16x16x32_bf16": 8, "32x32x2_f32": 18}    # matrix instruction (8 / 4 / 16 passes) -> anything else
REG = re.compile(r"(?<![\w.])([av])(?:(\d+)|\[(\d+):(\d+)\])(?!\w)")


def registers(text):
    """Set of (file, number) named by one operand."""
    return {(m[1], n) for m in REG.finditer(text) for n in range(int(m[2] or m[3]), int(m[2] or m[4]) + 1)}


class Instr:
    def __init__(self, text):
        self.text = text
        self.op, _, rest = text.partition(" ")
        ops = [registers(o) for o in rest.split(",")] if self.op[:2] != "s_" else []
        self.matrix = self.op.startswith("v_mfma")
        self.vector = self.op.startswith("v_") and not self.matrix
        self.named = set().union(*ops) if ops else set()
        self.sources = set().union(*ops[1:]) if self.matrix else set()
        both = "swap" in self.op
        self.writes = (self.named if both else ops[0]) if (self.vector or self.matrix) and ops else set()
        self.states = int(rest.split()[0], 0) + 1 if self.op == "s_nop" else 1
        self.preds = []


def kernels(dis):
    """(name, instructions with their predecessors) of every kernel in a disassembly."""
    for part in re.split(r"\n(?=[0-9a-f]{16} <)", dis):
        head = re.match(r"([0-9a-f]{16}) <(.+)>:\n", part)
        if not head or "\tv_mfma" not in part:
            continue
        code, at = [], {}
        for line in part[head.end():].splitlines():
            m = re.match(r"\s+(.+?)\s*// ([0-9A-F]+):", line)
            if m:
                at[int(m[2], 16)] = len(code)
                code.append((int(m[2], 16), Instr(m[1])))
        for i, (addr, ins) in enumerate(code):
            branch = re.match(r"s_c?branch\w* (\d+)", ins.text)
            if branch:
                off = int(branch[1])
                to = at.get(addr + 4 + 4 * (off - 65536 if off >= 32768 else off))
                assert to is not None, ins.text
                code[to][1].preds.append(i)
            if i + 1 < len(code) and ins.op not in ("s_branch", "s_endpgm"):
                code[i + 1][1].preds.append(i)
            assert ins.op not in ("s_setpc_b64", "s_swappc_b64"), "indirect branch"
        yield head[2], [ins for _, ins in code]


def too_close(code, i, limit, hit):
    """An instruction for which hit() holds and from which fewer than limit wait states pass until instruction i, on any path."""
    todo, seen = [(p, 0) for p in code[i].preds], {}
    while todo:
        j, passed = todo.pop()
        if seen.get(j, limit) <= passed:
            continue
        seen[j] = passed
        if hit(code[j], passed):
            return code[j]
        if passed + code[j].states < limit:
            todo += [(p, passed + code[j].states) for p in code[j].preds]
    return None


def hazards(code):
    wait = {ins.op: next(w for shape, w in RESULT_WAIT.items() if shape in ins.op) for ins in code if ins.matrix}
    for i, ins in enumerate(code):
        if ins.matrix:
            bad = too_close(code, i, OPERAND_WAIT, lambda o, _: o.vector and o.writes & ins.sources)
        elif ins.named:
            bad = too_close(code, i, max(wait.values()), lambda o, passed: o.matrix and passed < wait[o.op] and o.writes & ins.named)
        else:
            continue
        if bad:
            yield f"{bad.text}  ->  {ins.text}"


def disassembly(tmp_path):
    lib = tmp_path / "lib.so"
    lib.write_bytes(open(vb.LIB_PATH, "rb").read())
    subprocess.run([OBJDUMP, "--offloading", str(lib)], check=True, cwd=tmp_path, stdout=subprocess.DEVNULL)
    for f in sorted(tmp_path.glob("*gfx950")):
        yield subprocess.run([OBJDUMP, "-d", str(f)], check=True, capture_output=True, text=True).stdout


def test_checker_sees_a_missing_wait():
    text = "0000000000000000 <k>:\n" + "".join(f"\t{t} // {4 * i:012X}: 0\n" for i, t in enumerate([
        "v_mov_b32_e32 v4, 0", "s_nop 0", "v_mfma_f32_32x32x16_bf16 a[0:15], v[4:7], v[8:11], a[0:15]",
        "s_cbranch_scc0 1", "s_nop 15", "v_accvgpr_mov_b32 a20, a3", "s_endpgm"]))
    (_, code), = kernels(text)
    assert [h.split("  ->  ")[1].split()[0] for h in hazards(code)] == ["v_mfma_f32_32x32x16_bf16", "v_accvgpr_mov_b32"]


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
def test_no_matrix_instruction_misses_a_wait(tmp_path):
    if not os.path.exists(vb.LIB_PATH):
        build.build_lib(verbose=False)
    n, found = 0, []
    for dis in disassembly(tmp_path):
        for name, code in kernels(dis):
            n += sum(ins.matrix for ins in code)
            found += [f"{name}: {h}" for h in hazards(code)]
    assert n > 1000
    assert not found, f"{len(found)} of {n}: " + "\n".join(found[:20])
