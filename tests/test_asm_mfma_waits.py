"""Inline assembly beside matrix instructions.  The compiler inserts the wait
states that a matrix instruction (MFMA) needs after a vector write of its
operand, and that an access of its result needs after it, for instructions it
knows; statements of inline assembly it does not look into.  In the compiled
attention and decode kernels therefore:
  - two wait states or more lie between an inline write of a register and an
    MFMA that reads it (what the compiler keeps for its own writes);
  - no inline statement touches an MFMA's result registers while the MFMA may
    be in flight, that is before an instruction of the compiler's has accessed
    them (which it makes wait) or 20 wait states have passed."""
import pytest

from _asm import after, compile_to_asm, functions, operands, read, registers, written
from test_m0_guard import _hipcc

OPERAND_WAIT, RESULT_WAIT = 2, 20


def _faults(text):
    found, mfmas, inline = [], 0, 0
    for name, (code, labels) in functions(text).items():
        for i, ins in enumerate(code):
            if ins.inline and ins.op.startswith("v_"):
                inline += 1
                regs = written(ins)
                for j, n in after(code, labels, i, OPERAND_WAIT):
                    if code[j].op.startswith("v_mfma") and regs & read(code[j]):
                        found.append((name, n, ins.text, code[j].text))
            if ins.op.startswith("v_mfma"):
                mfmas += 1
                regs = registers(operands(ins.args)[0])
                walk = after(code, labels, i, RESULT_WAIT)
                stop = None
                while True:
                    try:
                        j, n = walk.send(stop)
                    except StopIteration:
                        break
                    touches = bool(regs & (written(code[j]) | read(code[j])))
                    if touches and code[j].inline:
                        found.append((name, n, ins.text, code[j].text))
                    # (a further MFMA on the same accumulator does not wait for the first)
                    stop = touches and not code[j].op.startswith("v_mfma")
    return found, mfmas, inline


@pytest.mark.skipif(_hipcc() is None, reason="hipcc not available")
@pytest.mark.parametrize("source", ["hifa4_attn.hip", "hifa4_decode.hip"])
def test_inline_assembly_keeps_the_mfma_waits(source, tmp_path):
    found, mfmas, inline = _faults(compile_to_asm(source, tmp_path))
    assert mfmas > 100 and inline > 100, "nothing to check: the assembly was not understood"
    assert not found, f"{len(found)} inline statements too close to an MFMA, for instance {found[0]}"


@pytest.mark.parametrize("lines,bad", [
    (["#ASMSTART", "v_mov_b32 v3, 1", "#ASMEND", "s_nop 0", "v_mfma_x v[8:11], v[0:3], v[4:5], 0"], True),
    (["#ASMSTART", "v_mov_b32 v3, 1", "#ASMEND", "s_nop 1", "v_mfma_x v[8:11], v[0:3], v[4:5], 0"], False),
    (["v_mov_b32 v3, 1", "v_mfma_x v[8:11], v[0:3], v[4:5], 0"], False),            # the compiler's own: it waits
    (["v_mfma_x v[8:11], v[0:3], v[4:5], 0", "s_nop 3", "#ASMSTART", "v_mov_b32 v9, v0", "#ASMEND"], True),
    (["v_mfma_x v[8:11], v[0:3], v[4:5], 0", "s_nop 3", "v_add_f32 v0, v8, v8", "#ASMSTART", "v_mov_b32 v9, v0",
      "#ASMEND"], False),
    (["#ASMSTART", "v_mov_b32 v3, 1", "#ASMEND", "s_cbranch_scc1 L1", "s_nop 7", "s_branch L2", "L1:",
      "v_mfma_x v[8:11], v[0:3], v[4:5], 0", "L2:", "s_endpgm"], True),              # along the branch
])
def test_the_check_sees_planted_code(lines, bad):
    assert bool(_faults("\n".join(["_Zf:"] + lines))[0]) == bad
