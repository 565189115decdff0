"""The built dk/dv kernel of head dimension 128, whose accumulating products are inline assembly: the
compiler does not know them for matrix instructions and adds no wait states around them.  What it placed
next to them is checked here in the built code."""
import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2606_30634_amd", "libasyncstage.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
SYMBOL = "_ZN12_GLOBAL__N_116flash_bwd_dkv128E8AttnArgs"
RESULT_STATES = 19  # wait states until anything but a matrix instruction may touch a 16-pass result
OPERAND_STATES = 2  # wait states from a vector instruction to the matrix instruction that reads its result


def _device_code(tmp):
    """The gfx950 code object of the library that holds SYMBOL."""
    data, at = open(LIB, "rb").read(), -1
    while (at := data.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 1)) >= 0:
        o = at + 32
        for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
            off, size, n = struct.unpack_from("<QQQ", data, o)
            o += 24 + n
            code = data[at + off:at + off + size]
            if SYMBOL.encode() in code:
                path = os.path.join(tmp, "code.elf")
                open(path, "wb").write(code)
                return path
    raise AssertionError("kernel not found in the library")


def _regs(text):
    out = set()
    for kind, lo, hi in re.findall(r"\b([av])\[?(\d+)(?::(\d+)\])?", text):
        out |= {(kind, r) for r in range(int(lo), int(hi or lo) + 1)}
    return out


class Insn:
    def __init__(self, line):
        text, _, rest = line.partition("//")
        self.op, _, args = text.strip().partition(" ")
        self.args = [a.strip() for a in re.split(r",(?![^\[]*\])", args)] if args else []
        self.addr = int(rest.strip().split(":")[0], 16)
        m = re.search(re.escape(SYMBOL) + r"(?:\+0x([0-9a-f]+))?>", rest)
        self.target = int(m.group(1) or "0", 16) if m and "branch" in self.op else None
        self.states = int(self.args[0], 0) + 1 if self.op == "s_nop" else 1
        self.mfma = self.op.startswith("v_mfma")
        self.touched = _regs(" ".join(self.args))
        vector = self.op.startswith("v_") and not self.mfma
        self.written = _regs(" ".join(self.args[:2 if "swap" in self.op else 1])) if vector else set()


def _check(seq, faults):
    """seq: instructions in the order they run."""
    for i, x in enumerate(seq):
        if not (x.mfma and x.args[0].startswith("a")):
            continue
        acc, operands = _regs(x.args[0]), _regs(" ".join(x.args[1:]))
        states = 0
        for y in reversed(seq[:i]):
            if states >= OPERAND_STATES:
                break
            if y.written & operands:
                faults.add(f"{y.op} {y.args} {states} states before {x.op} {x.args}")
            states += y.states
        states = 0
        for y in seq[i + 1:]:
            if states >= RESULT_STATES:
                break
            if y.touched & acc and not y.mfma:
                faults.add(f"{y.op} {y.args} {states} states after {x.op} {x.args}")
            states += y.states


@pytest.mark.skipif(not (os.path.exists(LIB) and os.path.exists(OBJDUMP)), reason="needs the built library and llvm-objdump")
def test_dkv128_accumulators_keep_their_distances(tmp_path):
    text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", f"--disassemble-symbols={SYMBOL}", _device_code(str(tmp_path))],
                          capture_output=True, text=True, check=True).stdout
    code = [Insn(l) for l in text.splitlines() if l.startswith("\t") and "// " in l]
    assert sum(x.mfma and x.args[0].startswith("a") for x in code) >= 64
    faults = set()
    _check(code, faults)
    base = {x.addr - code[0].addr: k for k, x in enumerate(code)}
    for k, x in enumerate(code):  # over each loop's end
        if x.target is not None and x.target in base and base[x.target] <= k:
            _check(code[max(0, k - 64):k + 1] + code[base[x.target]:base[x.target] + 64], faults)
    assert not faults, sorted(faults)[:8]
