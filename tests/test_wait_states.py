"""The built kernels keep the wait states between a matrix instruction and the vector instructions that read its result, on every path:
a walk over the disassembly of libaquakv.so from each v_mfma_f32_32x32x16_bf16 (8 passes: 12 states, which is what the compiler keeps on
the paths that it counts)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2501_19392_amd import binding as B

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
STATES = 12
OPERAND = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+))")
STORES = ("global_store", "ds_write", "buffer_store", "scratch_store", "flat_store")


def registers(text):
    out = set()
    for kind, first, last, one in OPERAND.findall(text):
        out.update((kind, i) for i in range(int(first or one), int(last or one) + 1))
    return out


def functions(listing):
    """(name, [(mnemonic, operands)], {label: index}) per function"""
    name, code, labels = None, [], {}
    for line in listing:
        if m := re.match(r"[0-9a-f]+ <(_Z\w+)>:", line):
            if name:
                yield name, code, labels
            name, code, labels = m[1], [], {}
        elif m := re.match(r"(?:[0-9a-f]+ )?<(L\d+)>:", line):
            labels[m[1]] = len(code)
        elif m := re.match(r"\s+([a-z]\w+)\s*(.*?)\s*(?://.*)?$", line):
            code.append((m[1], m[2]))
    if name:
        yield name, code, labels


def shortest(code, labels, start):
    """Wait states from the matrix instruction at `start` to the first read of its result, at most STATES are looked at."""
    result = registers(code[start][1].split(",")[0])
    best, seen, paths = STATES, {}, [(start + 1, 0)]
    while paths:
        at, w = paths.pop()
        while at < len(code) and w < best and seen.get(at, STATES) > w:
            seen[at] = w
            op, args = code[at]
            if op.startswith("v_mfma") or op == "s_endpgm":          # (matrix instructions wait for one another in hardware)
                if op == "s_endpgm":
                    break
            elif registers(args if op.startswith(STORES) else args.partition(",")[2]) & result:
                best = w
                break
            w += int(args, 0) + 1 if op == "s_nop" else 1
            target = labels[re.search(r"L\d+", args)[0]] if op == "s_branch" or op.startswith("s_cbranch") else None
            if op == "s_branch":
                at = target
                continue
            if target is not None:
                paths.append((target, w))
            at += 1
    return best


def test_results_of_matrix_instructions_are_not_read_early(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    shutil.copy(B.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    checked = 0
    for obj in sorted(tmp_path.glob("lib.so.*gfx950")):
        listing = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--symbolize-operands", str(obj)], check=True, capture_output=True,
                                 text=True).stdout.splitlines()
        for name, code, labels in functions(listing):
            for i, (op, _) in enumerate(code):
                if op == "v_mfma_f32_32x32x16_bf16":
                    checked += 1
                    assert shortest(code, labels, i) >= STATES, (name, i)
    assert checked > 1000
