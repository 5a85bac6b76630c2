"""Build libslim.so (the HIP kernels + C-ABI) in-tree with hipcc for gfx950."""
from __future__ import annotations

import glob
import os
import re
import subprocess
import sys
import tempfile

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libslim.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-munsafe-fp-atomics",
    # The prefill kernel addresses the accumulation registers by number from asm;
    # the compiler must not park spilled values there.
    "-mllvm", "-amdgpu-spill-vgpr-to-agpr=0",
    # m0 is a register the compiler keeps no value in; asm that writes it names it all the same, so that the
    # compiler's own uses stay in order with it, and would be warned about each time.
    "-Wall", "-Wno-unused-function", "-Wno-inline-asm",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


# Sources whose kernels address the accumulation registers by number (slim_mma.h).
FIXED_ACC_SOURCES = ("slim_gemm", "slim_gemm_sparse", "slim_lora_split")
_MATRIX_OP = re.compile(r"^\s*v_(mfma|smfmac)_")
_COMPILER_AGPR = re.compile(r"\ba\d+\b|\ba\[\d+:\d+\]")


def compiler_agpr_uses(asm_text: str) -> dict:
    """kernel -> instructions in which the compiler itself names an accumulation register.

    The hand-written asm of those sources spells single registers a[N] and only the matrix instructions
    take ranges; anything else (aN, or a range on a load or move) is the register allocator parking a
    value of its own there, where the kernel's matrix instructions will overwrite it."""
    out, name = {}, None
    for line in asm_text.splitlines():
        if line[:1] not in (" ", "\t", ""):
            head = line.split(":")[0]
            if line.rstrip().endswith(":") and not head.startswith("."):
                name = head
            continue
        code = line.split(";")[0]
        if name is None or not code.strip() or code.lstrip().startswith(".") or _MATRIX_OP.match(code):
            continue
        if _COMPILER_AGPR.search(code):
            out[name] = out.get(name, 0) + 1
    return out


# Instructions that read a register of another lane, and how many wait states after a vector instruction wrote it they may:
# the compiler sees to that between its own instructions, not where hand-written asm is one side of the pair.
_LANE_WAIT = 2
_LANE_READ = re.compile(r"\b(row_newbcast|row_share|row_shl|row_shr|row_ror|row_bcast|row_mirror|row_half_mirror|quad_perm|wave_\w+):?")
_VREG = re.compile(r"\bv(\d+)\b|\bv\[(\d+):(\d+)\]")


def _vregs(operand: str) -> set:
    out = set()
    for one, first, last in _VREG.findall(operand):
        out.update([int(one)] if one else range(int(first), int(last) + 1))
    return out


def lane_reads_too_early(asm_text: str) -> dict:
    """kernel -> instructions that read another lane's register less than two wait states after it was written, or that stand so
    near the start of an asm block that a copy the compiler puts right before the block would be."""
    out, name, recent, block = {}, None, [], None          # recent: (wait states, registers written); block: wait states since its start
    for line in asm_text.splitlines():
        if "ASMSTART" in line or "ASMEND" in line:
            block = 0 if "ASMSTART" in line else None
            continue
        if line[:1] not in (" ", "\t", ";", ""):
            head = line.split(":")[0]
            if line.rstrip().endswith(":") and not head.startswith("."):
                name = head
            continue
        code = line.split(";")[0].strip()
        if name is None or not code or code.startswith("."):
            continue
        op, _, rest = code.partition(" ")
        operands = rest.split(",")
        if op.startswith("v_permlane") and "swap" in op:
            read, written = _vregs(rest), _vregs(rest)
        else:
            read = _vregs(operands[1].strip().split(" ")[0]) if _LANE_READ.search(rest) and len(operands) > 1 else set()
            written = _vregs(operands[0]) if op.startswith("v_") and not _MATRIX_OP.match(" " + op) else set()
        near, waited = set(), 0
        for states, regs in reversed(recent):
            if waited >= _LANE_WAIT:
                break
            near |= regs
            waited += states
        if read & near or (read and block is not None and block < _LANE_WAIT):
            out[name] = out.get(name, 0) + 1
        states = int(operands[0], 0) + 1 if op == "s_nop" else 1
        recent = (recent + [(states, written)])[-_LANE_WAIT:]
        if block is not None:
            block += states
    return out


def build(verbose: bool = False) -> str:
    """Compile the library; the device assembly (a by-product of the same compilation) is checked for reads of other lanes' registers
    that come too early and, of the fixed-accumulator kernels, for accumulation registers used by the compiler."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *HIPCC_FLAGS, "-save-temps", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-o", LIB, *sources()]
    if verbose:
        print(" ".join(cmd), flush=True)
    with tempfile.TemporaryDirectory(prefix="slim_build_") as tmp:
        subprocess.run(cmd, check=True, cwd=tmp)
        for path in sorted(glob.glob(os.path.join(tmp, "*-hip-amdgcn-amd-amdhsa-gfx950.s"))):
            with open(path) as fh:
                bad = lane_reads_too_early(fh.read())
            if bad:
                os.remove(LIB)
                raise RuntimeError(f"{os.path.basename(path)}: registers of other lanes are read before what was written is there: {bad}")
        for stem in FIXED_ACC_SOURCES:
            with open(os.path.join(tmp, stem + "-hip-amdgcn-amd-amdhsa-gfx950.s")) as fh:
                bad = compiler_agpr_uses(fh.read())
            if bad:
                os.remove(LIB)
                raise RuntimeError(f"{stem}.hip: the compiler uses accumulation registers of kernels that address them "
                                   f"by number (their results would be overwritten): {bad}")
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    print(LIB)
    sys.exit(0)
