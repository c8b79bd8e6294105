"""gfx950 assembly of this library's own translation units, as control-flow
walkable code with the statements of inline assembly marked."""
import os
import re
import subprocess
from collections import namedtuple

from test_m0_guard import ROOT, _hipcc

Instr = namedtuple("Instr", "op args inline text")
_REG = re.compile(r"\b([va])(?:(\d+)|\[(\d+):(\d+)\])")
# no register result: the first operand is read
_NO_RESULT = ("s_", "v_cmp", "global_store", "buffer_store", "scratch_store", "ds_write", "global_load_lds")


def compile_to_asm(source, folder):
    out = os.path.join(str(folder), source + ".s")
    cmd = [_hipcc(), "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "--cuda-device-only", "-S", "-x", "hip",
           os.path.join(ROOT, "paper_2607_04302_amd", "csrc", source), "-o", out]
    subprocess.run(cmd, check=True, capture_output=True, timeout=600)
    with open(out) as f:
        return f.read()


def registers(text):
    out = set()
    for kind, one, first, last in _REG.findall(text):
        out.update((kind, i) for i in range(int(one or first), int(one or last) + 1))
    return out


def operands(args):
    return re.split(r",\s*(?![^\[]*\])", args)


def written(ins):
    return set() if ins.op.startswith(_NO_RESULT) else registers(operands(ins.args)[0])


def read(ins):
    if ins.op.startswith(_NO_RESULT):
        return registers(ins.args)
    return registers(",".join(operands(ins.args)[1:]))


def functions(text):
    """name -> (instructions, label -> index of the instruction after it)."""
    out, cur, labels, inline = {}, None, None, False
    for line in text.splitlines():
        if "#ASMSTART" in line or "#ASMEND" in line:
            inline = "#ASMSTART" in line
            continue
        s = line.split(";")[0].strip()
        label = re.match(r"([\w.$]+):$", s)
        if label and label.group(1).startswith("_Z"):
            cur, labels = [], {}
            out[label.group(1)] = cur, labels
        elif label and cur is not None:
            labels[label.group(1)] = len(cur)
        elif s and not s.startswith(".") and cur is not None:
            op, _, args = s.partition(" ")
            cur.append(Instr(op, args.strip(), inline, s))
    return out


def after(code, labels, start, limit):
    """Every instruction reachable within `limit` wait states of instruction
    `start`, with the wait states between the two.  Send True to go no further
    along a path."""
    def successors(i):
        op = code[i].op
        if op == "s_branch" or op.startswith("s_cbranch"):
            target = labels.get(operands(code[i].args)[-1])
            if target is not None:
                yield target
        if op not in ("s_branch", "s_endpgm", "s_setpc_b64"):
            yield i + 1

    todo, least = [(j, 0) for j in successors(start)], {}
    while todo:
        j, n = todo.pop()
        if j >= len(code) or n >= limit or least.get(j, limit) <= n:
            continue
        least[j] = n
        if (yield j, n):
            continue
        states = int(code[j].args, 0) + 1 if code[j].op == "s_nop" else 1
        todo += [(k, n + states) for k in successors(j)]
