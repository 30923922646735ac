"""Distances between matrix instructions and their operands, in the machine code of the library built here.
window_attn.hip spells P V of the persistent kernel out (mfma_acc), so the compiler keeps none of the distances that the
hardware does not enforce for them: they rest on the order of the slots and on mfma_settle."""
import os
import re

import pytest

from tests.test_scalar_loads import OBJDUMP, _kernels

# Wait states (an instruction is one, s_nop n is n + 1) that software keeps on gfx950, by the passes of the matrix
# instruction that wrote the register: until a vector or memory instruction reads or writes it, until another matrix
# instruction reads it as A or B, and as a C that is not just the register block written (the same block needs none).
# The compiler keeps these for the matrix instructions that it knows: 12, 5 and 18 are the nearest that occur here.
PASSES = {"v_mfma_f32_32x32x16_bf16": 8, "v_mfma_f32_32x32x2_f32": 16, "v_mfma_f32_4x4x4_16b_bf16": 2}
TO_VECTOR = TO_AB = {2: 5, 8: 12, 16: 18}               # (16: fp32)
TO_C = {2: 3, 8: 10, 16: 18}
VECTOR_TO_MATRIX = 2                                     # a vector write until a matrix instruction reads the register
EXEC_TO_MATRIX = 4
FAR = 20


def _regs(text):
    found = {(k, r) for k, a, b in re.findall(r"\b([va])\[(\d+):(\d+)\]", text) for r in range(int(a), int(b) + 1)}
    return found | {(k, int(r)) for k, r in re.findall(r"\b([va])(\d+)\b", text)}


class _Instruction:
    def __init__(self, text):
        self.text = text
        self.op, _, args = text.partition(" ")
        args = [a.strip() for a in args.split(",")]
        self.matrix = self.op.startswith("v_mfma") or self.op.startswith("v_smfma")
        self.vector = self.op.startswith("v_") and not self.matrix
        self.memory = self.op.startswith(("global_", "buffer_", "flat_", "scratch_", "ds_"))
        self.states = int(args[0], 0) + 1 if self.op == "s_nop" else 1
        self.all = set().union(*(_regs(a) for a in args))
        self.writes = set()
        if self.matrix:
            self.passes = PASSES[self.op]                # (a KeyError names a matrix instruction that needs its row above)
            self.writes, self.ab, self.c = _regs(args[0]), _regs(args[1]) | _regs(args[2]), _regs(args[3])
        elif self.vector:
            self.writes = _regs(args[0]) | (_regs(args[1]) if "swap" in self.op else set())


def _needed(first, then):
    """Wait states that `then` has to keep from `first` before it."""
    need = 0
    if first.matrix and then.matrix:
        if first.writes & then.ab:
            need = TO_AB[first.passes]
        if first.writes & then.c and first.writes != then.c:
            need = max(need, TO_C[first.passes])
    elif first.matrix and (then.vector or then.memory) and first.writes & then.all:
        need = TO_VECTOR[first.passes]
    elif first.vector and then.matrix:
        if first.writes & (then.ab | then.c):
            need = VECTOR_TO_MATRIX
        if first.op.startswith("v_cmpx"):
            need = EXEC_TO_MATRIX
    return need


def _too_near(body, labels):
    """(first, then, states between) of all pairs that stand nearer than they may, on any path."""
    code = [_Instruction(t) for t in body]
    before = [[i - 1] if i and not code[i - 1].op.startswith(("s_branch", "s_endpgm", "s_setpc")) else [] for i in range(len(code))]
    for i, c in enumerate(code):
        if c.op.startswith(("s_branch", "s_cbranch")):
            before[labels[c.text.split()[1]]].append(i)
    found = set()
    for i, c in enumerate(code):
        if not (c.matrix or c.vector or c.memory):
            continue
        todo, seen = [(j, 0) for j in before[i]], set()
        while todo:
            j, states = todo.pop()
            if (j, states) in seen or states >= FAR:
                continue
            seen.add((j, states))
            if states < _needed(code[j], c):
                found.add((code[j].text, c.text, states))
            todo += [(k, states + code[j].states) for k in before[j]]
    return sorted(found)


MFMA = "v_mfma_f32_32x32x16_bf16 a[0:15], v[0:3], v[4:7], a[0:15]"


@pytest.mark.parametrize("body,near", [
    (["v_cvt_pk_bf16_f32 v4, v8, v9", MFMA], True),
    (["v_cvt_pk_bf16_f32 v4, v8, v9", "s_nop 0", MFMA], True),
    (["v_cvt_pk_bf16_f32 v4, v8, v9", "s_nop 1", MFMA], False),
    (["v_permlane32_swap_b32_e32 v8, v5", MFMA], True),
    (["v_accvgpr_write_b32 a3, 0", MFMA], True),
    (["v_cmpx_gt_f32 exec, v8, v9", "s_nop 2", MFMA], True),
    ([MFMA, MFMA], False),                                             # the same block as C
    ([MFMA, "v_mfma_f32_32x32x16_bf16 a[0:15], v[0:3], v[4:7], a[8:23]"], True),
    ([MFMA, "s_nop 10", "v_accvgpr_read_b32 v8, a5"], True),
    ([MFMA, "s_nop 11", "v_accvgpr_read_b32 v8, a5"], False),
    ([MFMA, "s_nop 7", "ds_write_b128 v8, a[4:7]"], True),
    ([MFMA, "s_branch L0", "s_nop 15", "v_accvgpr_read_b32 v8, a5"], True),     # round the wait
])
def test_the_check_finds_what_stands_too_near(body, near):
    assert bool(_too_near(body, {"L0": len(body) - 1})) == near


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no ROCm disassembler")
def test_matrix_instructions_keep_their_distances(tmp_path):
    kernels = {k: v for k, v in _kernels(tmp_path).items() if "window_attn" in k}
    stream = [body for k, (body, _) in kernels.items() if "stream_kernel" in k]
    assert len(stream) == 2 and all(sum(i.startswith("v_mfma") and " a[" in i for i in body) >= 32 for body in stream)
    assert {k: near for k, (body, labels) in kernels.items() if (near := _too_near(body, labels))} == {}
