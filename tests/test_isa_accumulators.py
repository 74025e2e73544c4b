"""The large bf16 GEMM names its 256 accumulator registers in the text of its matrix instructions, unseen by the compiler. Looked
for in the disassembly of the built library (no GPU): any other use of that half of the register file in this kernel, results read
before the matrix instruction has written them, and operands that a vector instruction writes right before."""
import re
import shutil
import subprocess

import pytest

from paper_2605_10875_amd import sol
from test_isa_waits import OBJDUMP

MFMA_TO_READ = 18      # wait states from a matrix instruction (at most 16 passes) to a vector read of its result
VALU_TO_MFMA = 2       # wait states from a vector write to a matrix instruction that reads the register


def _regs(kind, text):
    out = set()
    for one, lo, hi in re.findall(r"\b%s(?:(\d+)\b|\[(\d+):(\d+)\])" % kind, text):
        out.update([int(one)] if one else range(int(lo), int(hi) + 1))
    return out


def _faults(lines):
    """(kernel, line, what) of every fault of the three kinds in k_gemm_mfma, and the number of its matrix instructions."""
    found, kernel, now, n = [], "", 0, 0
    made, written = {}, {}                    # accumulator register, vector register -> wait state of its last write
    for raw in lines:
        label = re.match(r"[0-9a-f]* ?<(.*)>:", raw)
        line = raw.split("//")[0].strip()
        if label:
            kernel, made, written = label.group(1), {}, {}
        if label or not line or "k_gemm_mfma" not in kernel:
            continue
        op, _, rest = line.partition(" ")
        now += int(rest.split()[0], 0) + 1 if op == "s_nop" else 1
        acc = _regs("a", rest)
        if op.startswith("v_mfma"):
            n += 1
            dst, src = rest.split(",", 1)
            if any(now - written.get(r, -99) <= VALU_TO_MFMA for r in _regs("v", src)):
                found.append((kernel, line, "operand just written"))
            made.update(dict.fromkeys(_regs("a", dst), now))
        elif op == "v_accvgpr_read_b32":
            if any(now - made.get(r, -99) <= MFMA_TO_READ for r in acc):
                found.append((kernel, line, "read too early"))
        elif acc:
            found.append((kernel, line, "another use of the accumulators"))
        if op.startswith("v_") and not op.startswith("v_mfma"):
            written.update(dict.fromkeys(_regs("v", rest.split(",")[0]), now))
    return found, n


def test_the_search_finds_each_fault():
    mfma = "\tv_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]"
    head, gap = ["<k_gemm_mfma>:"], ["\ts_nop 15", "\ts_nop 15"]
    assert _faults(head + [mfma] + gap + ["\tv_accvgpr_read_b32 v0, a3"]) == ([], 1)
    assert len(_faults(head + [mfma, "\tv_accvgpr_read_b32 v0, a3"])[0]) == 1
    assert len(_faults(head + ["\tv_accvgpr_write_b32 a7, v1"])[0]) == 1
    assert len(_faults(head + ["\tv_mov_b32_e32 v4, v9", mfma])[0]) == 1


@pytest.mark.skipif(OBJDUMP is None, reason="no llvm-objdump")
def test_the_accumulators_are_the_kernels_own(tmp_path):
    lib = shutil.copy(sol.lib_path(), tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", str(lib)], check=True, capture_output=True, cwd=tmp_path)
    total = 0
    for p in (p for p in tmp_path.iterdir() if p.name.endswith("gfx950")):
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(p)], check=True, capture_output=True, text=True).stdout
        found, n = _faults(text.splitlines())
        total += n
        assert not found, (len(found), found[:3])
    assert total > 0
