"""The large bf16 GEMM names its 256 accumulator registers in the text of its matrix instructions, unseen by the compiler. Looked
for in the disassembly of the built library (no GPU): any other use of that half of the register file in this kernel, results read
before the matrix instruction has written them, and operands that a vector instruction writes right before."""
import os
import shutil
import subprocess

import pytest

from paper_2605_10875_amd import build, isa, sol
from paper_2605_10875_amd.isa import accumulator_faults as _faults
from test_isa_waits import OBJDUMP

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


@pytest.fixture
def objects_to_link(tmp_path, monkeypatch):
    """A build whose objects are there already, in a folder of its own."""
    monkeypatch.setattr(build, "OBJ", str(tmp_path))
    monkeypatch.setattr(build, "LIB", str(tmp_path / "libsol.so"))
    monkeypatch.setattr(build, "_compile", lambda src, verbose: open(build._obj(src), "w").close())
    return tmp_path


@pytest.mark.parametrize("listing", ["<k_gemm_mfma>:\n\tv_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], 0\n\tv_accvgpr_write_b32 a7, v1",
                                     "<k_gemm_tile>:\n\tv_mov_b32_e32 v4, v9"], ids=["other_use", "kernel_not_there"])
def test_the_build_stops_where_the_search_does(objects_to_link, monkeypatch, listing):
    monkeypatch.setattr(isa, "device_code", lambda path: [listing])
    with pytest.raises(RuntimeError, match="k_gemm_mfma"):
        build.build(force=True)
    assert not os.path.exists(build.LIB)


def test_the_build_stops_without_the_disassembler(objects_to_link, monkeypatch):
    monkeypatch.setattr(isa, "objdump", lambda: None)
    with pytest.raises(RuntimeError, match="llvm-objdump"):
        build.build(force=True)
    assert not os.path.exists(build.LIB)
