"""Wait states around the library's inline assembly, read off the compiler's assembly of every kernel (no GPU).

The compiler keeps the distance that a matrix instruction's registers need from the vector instructions after it, but only for
instructions it selects itself: inline assembly is text to it.  For v_mfma_*_16x16x64_i8 on gfx950 (four passes) these are 8 wait states
before another instruction reads or overwrites its result, and 3 before one overwrites its C operand; a load whose scalar base
address a vector instruction wrote needs 5.  An instruction counts as one wait state, s_nop N as N + 1."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2007_12216_amd.build import compile_command

RESULT, C_OPERAND, SCALAR_BASE = 8, 3, 5


def registers(text, letter):
    out = set()
    for lo, hi, one in re.findall(r"\b%s\[(\d+):(\d+)\]|\b%s(\d+)\b" % (letter, letter), text):
        out |= {int(one)} if one else set(range(int(lo), int(hi) + 1))
    return out


def functions(path):
    """{name: (instructions, {label: index})}, an instruction as (mnemonic, operands, inside inline assembly, text)."""
    out, code, labels, inline = {}, None, None, False
    for line in open(path):
        start = re.match(r"(_Z\w+):", line)
        if start:
            code, labels, inline = [], {}, False
            out[start.group(1)] = (code, labels)
        if code is None or start:
            continue
        line = line.strip()
        if "ASMSTART" in line or "ASMEND" in line:
            inline = "ASMSTART" in line
            continue
        label = re.match(r"(\.L\w+):", line)
        if label:
            labels[label.group(1)] = len(code)
        text = line.split(";")[0].strip()
        if text and not text.startswith(".") and not text.endswith(":"):
            op, _, rest = text.partition(" " if " " in text and "\t" not in text else "\t")
            operands = [o.strip() for o in re.split(r",\s*(?![^\[]*\])", rest)]
            code.append((op, operands, inline, text))
    return out


def violations(code, labels):
    """Inline-assembly instructions that come too soon, on any path."""
    found = []
    for at, (op, operands, _, text) in enumerate(code):
        scalar = op in ("v_readfirstlane_b32", "v_readlane_b32")
        if not (op.startswith("v_mfma") or scalar):
            continue
        result = frozenset() if scalar else frozenset(registers(operands[0], "v"))
        c_operand = frozenset() if scalar else frozenset(registers(operands[3], "v") - result)
        base = frozenset(registers(operands[0], "s")) if scalar else frozenset()
        paths, seen = [(at + 1, 0, result, c_operand, base)], {}
        while paths:
            i, waited, d, c, s = paths.pop()
            if i >= len(code) or waited >= RESULT or not (d or c or s) or seen.get((i, d, c, s), 99) <= waited:
                continue
            seen[i, d, c, s] = waited
            op2, operands2, inline, text2 = code[i]
            if op2 == "s_endpgm":
                continue
            if op2 == "s_branch" or op2.startswith("s_cbranch"):
                paths.append((labels[operands2[0]], waited + 1, d, c, s))
                if op2 == "s_branch":
                    continue
            writes, reads = set(), set()
            if op2.startswith("v_"):
                writes = registers(operands2[0], "v")
                reads = set().union(*[registers(o, "v") for o in operands2[1:]])
            elif inline and not op2.startswith("s_"):
                reads = set().union(*[registers(o, "v") for o in operands2])
                if waited < SCALAR_BASE and any(registers(o, "s") & s for o in operands2):
                    found.append((text, text2, "scalar base", waited))
            if inline and not op2.startswith("v_mfma"):
                if (reads | writes) & d:
                    found.append((text, text2, "result", waited))
                if writes & c and waited < C_OPERAND:
                    found.append((text, text2, "C operand", waited))
            if op2.startswith("s_") and operands2:
                s = s - registers(operands2[0], "s")
            paths.append((i + 1, waited + (int(operands2[0], 0) + 1 if op2 == "s_nop" else 1), d - writes, c - writes, s))
    return found


PLANTED = {
    "result": "v_mfma_i32_16x16x64_i8 v[0:3], v[8:11], v[12:15], v[4:7]\n\ts_nop 6\n\t;;#ASMSTART\n\tv_mad_u32_u24 v20, s0, v1, v20\n\t;;#ASMEND",
    "C operand": "v_mfma_i32_16x16x64_i8 v[0:3], v[8:11], v[12:15], v[4:7]\n\ts_nop 1\n\t;;#ASMSTART\n\tv_mul_lo_u32 v4, s0, v20\n\t;;#ASMEND",
    "scalar base": "v_readfirstlane_b32 s4, v1\n\ts_nop 3\n\t;;#ASMSTART\n\tglobal_load_lds_dwordx4 v2, s[4:5]\n\t;;#ASMEND",
}


@pytest.mark.parametrize("what", sorted(PLANTED))
def test_the_walk_sees_an_instruction_that_comes_too_soon(tmp_path, what):
    for nops, expected in ((0, [what]), (1, [])):
        path = tmp_path / "planted.s"
        path.write_text("_Zplanted:\n\t" + PLANTED[what].replace("\t;;#ASMSTART", "\ts_nop 0\n" * nops + "\t;;#ASMSTART") + "\n\ts_endpgm\n")
        (code, labels), = functions(path).values()
        assert [v[2] for v in violations(code, labels)] == expected


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not available")
def test_inline_assembly_keeps_the_wait_states_of_matrix_results(tmp_path):
    path = str(tmp_path / "rnswino.s")
    source = [a for a in compile_command(path) if not a.endswith("plan_math.cpp") and a != "-shared"]
    build = subprocess.run(source + ["-S", "--cuda-device-only"], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert build.returncode == 0, build.stdout
    kernels = functions(path)
    assert sum(inline for code, _ in kernels.values() for _, _, inline, _ in code) > 1000
    found = {name: v for name, (code, labels) in kernels.items() for v in [violations(code, labels)] if v}
    assert not found, "\n".join(f"{name}: {v[0]} ({len(v)} in all)" for name, v in found.items())
