"""Scalar loads of the attention kernels, in the machine code of the library built here: window_attn.hip issues some by
inline assembly, and the compiler neither knows that their registers are still to be written nor waits for them."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2604_06036_amd import binding

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def _kernels(tmp_path):
    """name -> (instructions, {label: index of its instruction}) of every kernel in the library."""
    lib = shutil.copy(binding.LIB_PATH, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=tmp_path, check=True, capture_output=True)
    kernels, body, labels = {}, None, None
    for code in sorted(f for f in os.listdir(tmp_path) if f.endswith("gfx950")):
        text = subprocess.run([OBJDUMP, "-d", "--symbolize-operands", code], cwd=tmp_path, check=True, capture_output=True, text=True)
        for line in text.stdout.splitlines():
            line = line.split("//")[0].strip()
            name, label = re.match(r"[0-9a-f]+ <(\w+)>:$", line), re.match(r"<(L\d+)>:$", line)
            if name and not re.match(r"L\d+$", name.group(1)):
                body, labels = [], {}
                kernels[name.group(1)] = body, labels
            elif name or label:
                labels[(name or label).group(1)] = len(body)
            elif body is not None and line and not line.startswith("Disassembly"):
                body.append(line)
    return kernels


def _sgprs(text):
    spans = [(int(a), int(b)) for a, b in re.findall(r"\bs\[(\d+):(\d+)\]", text)]
    spans += [(int(a), int(a)) for a in re.findall(r"\bs(\d+)\b", text)]
    return {r for a, b in spans for r in range(a, b + 1)}


def _unwaited(body, labels):
    """Instructions that touch a register a scalar load has yet to write, or end the wave before it has, on any path."""
    seen, todo, found = [None] * len(body), [(0, frozenset())], set()
    while todo:
        i, pending = todo.pop()
        while seen[i] is None or not pending <= seen[i]:
            pending = seen[i] = pending | (seen[i] or frozenset())
            op, _, args = body[i].partition(" ")
            if pending & _sgprs(args) or (op == "s_endpgm" and pending):
                found.add((i, body[i]))
            if op.startswith(("s_load", "s_buffer_load")):
                pending = pending | _sgprs(args.split(",")[0])
            elif op == "s_waitcnt" and "lgkmcnt(0)" in args:
                pending = frozenset()
            elif op == "s_endpgm":
                break
            elif op == "s_branch" or op.startswith("s_cbranch"):
                target = labels[args.split()[0]]
                if op == "s_branch":
                    i = target
                    continue
                todo.append((target, pending))
            i += 1
    return sorted(found)


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no ROCm disassembler")
def test_every_scalar_load_is_waited_for(tmp_path):
    kernels = {k: v for k, v in _kernels(tmp_path).items() if "window_attn" in k}
    assert sum("tile_kernel" in k for k in kernels) >= 5 and any("stream_kernel" in k for k in kernels)
    assert all(any(i.startswith("s_load") for i in body) for body, _ in kernels.values())
    assert {k: found for k, (body, labels) in kernels.items() if (found := _unwaited(body, labels))} == {}
