"""The grouped GEMM issues its MFMAs from inline asm, which the compiler does not know to be MFMAs: it inserts no wait
states around them.  The source keeps everything else away from their operands (pin(), settle()), but where the
compiler puts register moves cannot be said in C++, so the built kernels are read: along every path, an MFMA result is not
touched by anything but an MFMA that accumulates into it for 19 wait states (the most any MFMA of gfx950 needs), and no MFMA
operand is written by a vector instruction in the two wait states before it."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2501_10375_amd import moe

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
RESULT_WAIT, OPERAND_WAIT = 19, 2


def registers(operand):
    m = re.fullmatch(r"\|?-?([va])(?:(\d+)|\[(\d+):(\d+)\])\|?", operand.strip())
    if not m:
        return frozenset()
    lo, hi = (m.group(2), m.group(2)) if m.group(2) else (m.group(3), m.group(4))
    return frozenset((m.group(1), i) for i in range(int(lo), int(hi) + 1))


class Instruction:
    def __init__(self, line):
        code, _, comment = line.partition("//")
        op, _, rest = code.strip().partition(" ")
        self.op, self.text = op, code.strip()
        self.address = int(comment.split(":")[0], 16)
        operands = re.findall(r"[^,\[\s]*\[[^\]]*\]|[^,\s]+", rest)
        self.regs = [registers(o) for o in operands]
        self.mfma = op.startswith("v_mfma")
        self.wait = int(rest) + 1 if op == "s_nop" else 1
        target = re.search(r"\+0x([0-9a-f]+)>", comment)
        self.target = int(target.group(1), 16) if op.startswith(("s_branch", "s_cbranch")) and target else None
        vector = op.startswith("v_") and not self.mfma
        both = "swap" in op
        self.vector_writes = frozenset().union(*(self.regs if both else self.regs[:1])) if vector and self.regs else frozenset()
        self.touches = frozenset().union(*self.regs) if self.regs else frozenset()


def parse(text, wanted):
    """{kernel: instructions} of a disassembly."""
    kernels, current = {}, None
    for line in text.splitlines():
        m = re.match(r"([0-9a-f]+) <(\S+)>:", line)
        if m:
            current = m.group(2) if wanted in m.group(2) else None
            if current:
                kernels[current] = []
        elif current and "//" in line and line.startswith("\t"):
            kernels[current].append(Instruction(line))
    return kernels


def hazards(code):
    """(where, what) of every pair that lies too close on some path."""
    at = {c.address: n for n, c in enumerate(code)}
    base = code[0].address

    def follow(n, waits):
        """Instructions reachable from behind `n`, with fewer than `waits` wait states in between."""
        todo, seen = [(n, waits)], {}
        while todo:
            i, left = todo.pop()
            if i != n or left != waits:
                left -= code[i].wait
            if left <= 0 and not (i == n and left == waits):
                continue
            nxt = [] if code[i].op in ("s_branch", "s_endpgm") else [i + 1]
            if code[i].target is not None:
                nxt.append(at[base + code[i].target])
            for j in nxt:
                if j < len(code) and seen.get(j, 0) < left:
                    seen[j] = left
                    todo.append((j, left))
        return seen

    found = []
    for n, c in enumerate(code):
        if c.mfma:
            result = c.regs[0]
            for j in follow(n, RESULT_WAIT):
                o = code[j]
                accumulates = o.mfma and o.regs[0] == result and o.regs[3] == result and not (result & (o.regs[1] | o.regs[2]))
                if result & o.touches and not accumulates:
                    found.append((c.text, o.text))
        elif c.vector_writes:
            for j in follow(n, OPERAND_WAIT):
                if code[j].mfma and c.vector_writes & code[j].touches:
                    found.append((c.text, code[j].text))
    return found


def listing(*lines):
    return "0000000000000100 <k>:\n" + "".join(f"\t{l} // {0x100 + 4 * i:012X}: 00000000\n" for i, l in enumerate(lines))


MFMA = "v_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]"


@pytest.mark.parametrize("lines,bad", [
    ((MFMA, MFMA, "s_nop 15", "s_nop 15", "v_accvgpr_read_b32 v9, a3"), 0),
    ((MFMA, "s_nop 15", "v_accvgpr_read_b32 v9, a3"), 1),
    ((MFMA, "global_store_dwordx4 v[10:11], a[0:3], off"), 1),
    (("v_accvgpr_write_b32 a0, 0", "s_nop 1", MFMA), 0),
    (("v_accvgpr_write_b32 a0, 0", "s_nop 0", MFMA), 1),
    (("v_mov_b32_e32 v5, v20", MFMA), 1),
    (("v_mov_b32_e32 v8, v20", MFMA), 0),
    ((MFMA, "v_mfma_f32_16x16x32_bf16 a[4:7], a[0:3], v[4:7], a[4:7]"), 1),
])
def test_the_reader_finds_what_lies_too_close(lines, bad):
    assert len(hazards(parse(listing(*lines), "k")["k"])) == bad


def test_the_reader_follows_branches():
    text = ("0000000000000100 <k>:\n\tv_mov_b32_e32 v5, v20 // 000000000100: 0\n"
            f"\t{MFMA} // 000000000104: 0\n\ts_nop 15 // 000000000108: 0\n\ts_nop 15 // 00000000010C: 0\n"
            "\tv_mov_b32_e32 v0, v30 // 000000000110: 0\n\ts_cbranch_scc1 65532 // 000000000114: 0 <k+0x4>\n"
            "\ts_endpgm // 000000000118: 0\n")
    assert len(hazards(parse(text, "k")["k"])) == 2  # the move in front, and the one before the jump back


def test_built_grouped_gemm_kernels_have_no_mfma_hazard(tmp_path):
    if not os.path.exists(OBJDUMP) or not os.path.exists(moe.LIB_PATH):
        pytest.skip("needs llvm-objdump and the built library")
    shutil.copy(moe.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, check=True, stdout=subprocess.DEVNULL)
    kernels = {}
    for name in sorted(os.listdir(tmp_path)):
        if "gfx950" in name:
            text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", name], cwd=tmp_path, check=True, text=True,
                                  stdout=subprocess.PIPE).stdout
            kernels.update(parse(text, "grouped_gemm_kernel"))
    assert len(kernels) >= 5
    for name, code in kernels.items():
        assert sum(c.mfma for c in code) > 1000, name
        assert hazards(code) == [], name
