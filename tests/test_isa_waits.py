"""Wait states around hand-written vector instructions, looked for in the disassembly of the built library (no GPU).

On gfx950 a scalar register that a vector instruction has written may be read by another vector instruction only after two
more wait states, by a memory instruction (as its base address) after five. The compiler keeps these distances between
instructions of its own; the inside of an inline-asm block it does not look at, and the loads that go straight to the LDS are
inline asm with a scalar base."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2605_10875_amd import sol

OBJDUMP = next((p for p in ("/opt/rocm/llvm/bin/llvm-objdump", shutil.which("llvm-objdump")) if p and os.path.exists(p)), None)
WAIT_STATES = 2
MEMORY_WAIT_STATES = 5


def _sgprs(operand):
    m = re.fullmatch(r"[-|]*s(\d+)\|?", operand)
    if m:
        return {int(m.group(1))}
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    return set(range(int(m.group(1)), int(m.group(2)) + 1)) if m else set()


def _early_reads(lines, readers=("v_",), wait_states=WAIT_STATES):
    """(kernel, writing line, reading line) of every read of a scalar register, by instructions that begin with one of `readers`, less than
    wait_states after a vector instruction has written it."""
    found, kernel, written = [], "", {}               # written: register -> (wait states since, line)
    for raw in lines:
        label = re.match(r"[0-9a-f]* ?<(.*)>:", raw)
        line = raw.split("//")[0].strip()
        if label or not line:
            kernel, written = (label.group(1), {}) if label else (kernel, written)
            continue
        op, _, rest = line.partition(" ")
        operands = [t.split()[0] for t in rest.split(",") if t.strip()]
        if op == "s_nop":
            written = {r: (n + int(operands[0], 0) + 1, w) for r, (n, w) in written.items()}
            continue
        if op.startswith(readers):
            sources = operands[2 if "_co_" in op or "div_scale" in op else 1 if op.startswith("v_") else 0:]      # (these write a mask as their second operand)
            for r in set().union(*map(_sgprs, sources)):
                if r in written and written[r][0] < wait_states:
                    found.append((kernel, written[r][1], line))
        written = {r: (n + 1, w) for r, (n, w) in written.items() if n + 1 < wait_states}
        if op.startswith(("v_readlane", "v_readfirstlane", "v_cmp")) and operands:
            written.update({r: (0, line) for r in _sgprs(operands[0])})
    return found


def test_the_search_for_early_reads_finds_one():
    bad = ["<k>:", "\tv_readlane_b32 s9, v14, s2", "\tv_writelane_b32 v14, s9, 16"]
    assert len(_early_reads(bad)) == 1
    assert not _early_reads(bad[:2] + ["\ts_nop 1"] + bad[2:])


def test_the_search_for_early_bases_finds_one():
    memory = dict(readers=("global_", "buffer_", "flat_", "scratch_"), wait_states=MEMORY_WAIT_STATES)
    bad = ["<k>:", "\tv_readlane_b32 s9, v14, 2", "\ts_add_u32 m0, s4, s5", "\ts_nop 0", "\tglobal_load_lds_dwordx4 v3, s[8:9]"]
    assert len(_early_reads(bad, **memory)) == 1
    assert not _early_reads(bad[:2] + ["\ts_nop 2"] + bad[2:], **memory)


@pytest.mark.skipif(OBJDUMP is None, reason="no llvm-objdump")
def test_no_scalar_register_is_read_too_early(tmp_path):
    lib = shutil.copy(sol.lib_path(), tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", str(lib)], check=True, capture_output=True, cwd=tmp_path)
    objects = sorted(p for p in tmp_path.iterdir() if p.name.endswith("gfx950"))
    assert objects
    for p in objects:
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(p)], check=True, capture_output=True, text=True).stdout
        found = _early_reads(text.splitlines())
        found += _early_reads(text.splitlines(), ("global_", "buffer_", "flat_", "scratch_"), MEMORY_WAIT_STATES)
        assert not found, (len(found), found[:3])
