"""What the compiler does not check in the library's own machine code, looked for in its disassembly (no GPU).

The large bf16 GEMM (k_gemm_mfma) names its 256 accumulator registers in the text of its matrix instructions. To the compiler they
are scratch: another compiler, or another epilogue, could put values of its own into them and the sums would be wrong without an
error. So build.py runs this search over every object that it links, and fails on a hit."""
import os
import re
import shutil
import subprocess
import tempfile

MFMA_TO_READ = 18      # wait states from a matrix instruction (at most 16 passes) to a vector read of its result
VALU_TO_MFMA = 2       # wait states from a vector write to a matrix instruction that reads the register


def objdump():
    """Path of llvm-objdump, None if there is none."""
    roots = [r for r in (os.environ.get("ROCM_PATH"), "/opt/rocm") if r]
    here = [os.path.join(r, "llvm", "bin", "llvm-objdump") for r in roots]
    return next((p for p in here if os.path.exists(p)), None) or shutil.which("llvm-objdump")


def device_code(path):
    """Disassembly of each gfx950 code object inside an object file or library."""
    tool = objdump()
    if tool is None:
        raise RuntimeError("no llvm-objdump: the accumulators of k_gemm_mfma cannot be checked")
    with tempfile.TemporaryDirectory() as tmp:
        here = shutil.copy(path, os.path.join(tmp, "object"))
        subprocess.run([tool, "--offloading", here], check=True, capture_output=True, cwd=tmp)
        return [subprocess.run([tool, "-d", "--no-show-raw-insn", os.path.join(tmp, n)], check=True, capture_output=True, text=True).stdout
                for n in sorted(os.listdir(tmp)) if n.endswith("gfx950")]


def _regs(kind, text):
    out = set()
    for one, lo, hi in re.findall(r"\b%s(?:(\d+)\b|\[(\d+):(\d+)\])" % kind, text):
        out.update([int(one)] if one else range(int(lo), int(hi) + 1))
    return out


def accumulator_faults(lines):
    """(kernel, line, what) of every other use of the accumulator registers in k_gemm_mfma, of results read before the matrix
    instruction has written them and of operands that a vector instruction writes right before; and the number of its matrix
    instructions."""
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


def check_accumulators(paths):
    """Raises if the search finds anything in these files, or no k_gemm_mfma at all."""
    total = 0
    for path in paths:
        for text in device_code(path):
            found, n = accumulator_faults(text.splitlines())
            total += n
            if found:
                raise RuntimeError(f"{os.path.basename(path)}: k_gemm_mfma: {len(found)} faults, the first: {found[:3]}")
    if total == 0:
        raise RuntimeError("no matrix instruction of k_gemm_mfma in " + ", ".join(map(os.path.basename, paths)))
