"""Build of the HIP library libscalify.so for gfx950 (MI355X).

Every .hip source under csrc/ is compiled by hipcc in parallel and linked into
one shared library next to this file. Packed-fp32 instructions are disabled
for all device code.

The GEMM kernels with many accumulators keep them in AGPRs that only their
inline asm names (AccTile in csrc/gemm_kernel.h); the compiler does not know
these registers hold values. The build therefore disassembles the objects of
these kernels and fails if, in any kernel that uses those accumulators, any
instruction other than the accumulator asm's own forms (an MFMA whose
destination and C operand are the same a[n:n+3], a write of 0, a read into a
VGPR) names one of them -- the compiler spilling into it or using it as the
data of a load or an MFMA operand.

No GEMM kernel may use scratch memory, but for the fused epilogue of the 8-wave
kernel (gemm_*_fused), which holds accumulators, residual codes and channel
exponents at once and keeps some of them there.

The loads of these kernels are inline asm too, so the compiler does not keep
the distance their scalar operands need: the build fails if a vector memory
instruction reads a scalar register that a vector instruction wrote less than
five wait states before.
"""
from __future__ import annotations

import concurrent.futures as cf
import glob
import os
import re
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libscalify.so")
ARCH = "gfx950"

HIPCC_FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument", "-Wno-pass-failed",
]


def _hipcc() -> str:
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return os.path.join(rocm, "bin", "hipcc")


def _llvm(tool: str) -> str:
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return os.path.join(rocm, "llvm", "bin", tool)


_KERNEL = re.compile(r"^[0-9a-f]+ <(\S+)>:$")
_AGPR_MFMA = re.compile(r"v_mfma\S* a\[")
_ANY_AGPR = re.compile(r"\ba\d+\b|\ba\[\d+:\d+\]")
# The only instructions that may name an AGPR in a kernel whose accumulators
# the inline asm holds: the asm's MFMA on an accumulator tile (destination and
# C operand the same a[n:n+3]), its zeroing write and its read into a VGPR.
_ASM_MFMA = re.compile(r"^v_mfma\S*\s+(a\[\d+:\d+\]),\s*v\[\d+:\d+\],\s*v\[\d+:\d+\],\s*(a\[\d+:\d+\])")
_ASM_ZERO = re.compile(r"^v_accvgpr_write_b32\s+a\d+,\s*0\s*$")
_ASM_READ = re.compile(r"^v_accvgpr_read_b32\s+v\d+,\s*a\d+\s*$")


def _asm_agpr_form(insn: str) -> bool:
    """Whether an instruction that names an AGPR is one of the accumulator
    asm's own forms."""
    m = _ASM_MFMA.match(insn)
    if m:
        # the MFMA's remaining operands (block-scale words, modifiers) name no AGPR
        rest = insn[m.end():]
        return m.group(1) == m.group(2) and not _ANY_AGPR.search(rest)
    return bool(_ASM_ZERO.match(insn) or _ASM_READ.match(insn))


def _sgprs(text: str) -> set:
    """The scalar registers a piece of an instruction names."""
    regs = set()
    for m in re.finditer(r"\bs(\d+)\b|\bs\[(\d+):(\d+)\]", text):
        lo, hi = (m.group(1),) * 2 if m.group(1) else (m.group(2), m.group(3))
        regs.update(range(int(lo), int(hi) + 1))
    return regs


def scalar_distance_violations(insns) -> list:
    """Vector memory instructions that read a scalar register less than five
    wait states after a vector instruction wrote it (straight-line scan)."""
    bad, recent = [], []
    for insn in insns:
        if not insn:
            continue
        op = insn.split()[0]
        if op.startswith(("buffer_", "global_", "flat_", "scratch_")):
            used = _sgprs(insn)
            if any(age < 5 and used & regs for age, regs in recent):
                bad.append(insn)
        step = int(insn.split()[1]) + 1 if op == "s_nop" else 1
        recent = [(age + step, regs) for age, regs in recent if age + step < 5]
        if op.startswith("v_") and " " in insn:
            regs = _sgprs(insn.split(None, 1)[1].split(",")[0])
            if regs:
                recent.append((0, regs))
    return bad


def _agprs(insn: str) -> set:
    """The AGPR numbers an instruction names."""
    regs = set()
    for m in re.finditer(r"\ba(\d+)\b|\ba\[(\d+):(\d+)\]", insn):
        lo, hi = (m.group(1),) * 2 if m.group(1) else (m.group(2), m.group(3))
        regs.update(range(int(lo), int(hi) + 1))
    return regs


_MID_KERNEL = re.compile(r"mid_gemm_kernelILb[01]ELb[01]ELi\d+ELi\d+ELi(\d+)ELi\d+EEE")


def pinned_kernel(src: str, name: str) -> bool:
    """Whether a kernel of this source that multiplies into AGPRs keeps its
    accumulators in asm-named ones: every such kernel of the gemm_* sources,
    and of the mid_* sources those with 256 columns (8 accumulator tiles per
    row of tiles); the others leave their accumulators to the compiler."""
    base = os.path.basename(src)
    if base.startswith("gemm_"):
        return True
    if base.startswith("mid_"):
        m = _MID_KERNEL.search(name)
        if not m:
            raise RuntimeError(f"{base}: which accumulators does {name} hold? (its name has another form)")
        return m.group(1) == "8"
    return False


def check_code(obj: str, tmp: str) -> int:
    """Disassemble the gfx950 code of one object and check every kernel that
    keeps accumulators in asm-named AGPRs, and every function's scalar
    operands of vector memory. Returns the number of kernels with such
    accumulators; raises RuntimeError on a violation."""
    base = os.path.join(tmp, os.path.basename(obj))
    subprocess.run([_llvm("llvm-objcopy"), f"--dump-section=.hip_fatbin={base}.fatbin", obj],
                   check=True, capture_output=True)
    subprocess.run([_llvm("clang-offload-bundler"), "--unbundle", "--type=o",
                    f"--input={base}.fatbin", f"--targets=hipv4-amdgcn-amd-amdhsa--{ARCH}",
                    f"--output={base}.co"], check=True, capture_output=True)
    dis = subprocess.run([_llvm("llvm-objdump"), "-d", f"--mcpu={ARCH}", f"{base}.co"],
                         check=True, capture_output=True, text=True).stdout
    kernels = {}
    name = None
    for line in dis.splitlines():
        m = _KERNEL.match(line)
        if m:
            name = m.group(1)
            kernels[name] = []
        elif name is not None:
            kernels[name].append(line)
    return check_functions(obj, kernels)


def check_functions(obj: str, kernels: dict) -> int:
    """The checks of check_code on disassembled functions: name -> lines."""
    base = os.path.basename(obj).split(".")[0]
    checked = 0
    for name, body in kernels.items():
        insns = [line.split("//")[0].strip() for line in body]
        near = scalar_distance_violations(insns)
        if near:
            raise RuntimeError(f"{obj}: {name} reads a scalar register too soon: {near[:4]}")
        spills = [l for l in insns if l.startswith("scratch_")]
        if spills and not base.endswith("_fused"):
            raise RuntimeError(f"{obj}: {name} uses scratch memory: {spills[:4]}")
        if not any(_AGPR_MFMA.search(l) for l in insns):
            # Out-of-line functions that the kernels call while accumulators
            # still sit in AGPRs must leave AGPRs alone.
            bad = [l for l in insns if _ANY_AGPR.search(l)]
            if bad and base.startswith("gemm_"):
                raise RuntimeError(f"{obj}: function {name} uses AGPRs: {bad[:4]}")
            continue
        if not pinned_kernel(obj, name):
            continue
        checked += 1
        held = set()
        for insn in insns:
            if _AGPR_MFMA.search(insn):
                held |= _agprs(insn)
        bad = [insn for insn in insns if _agprs(insn) & held and not _asm_agpr_form(insn)]
        if bad:
            raise RuntimeError(f"{obj}: kernel {name} has compiler-placed AGPR accesses next to the "
                               f"asm-held accumulators: {bad[:4]}")
    # (of the mid_* sources, one kernel with 256 columns for each pair of formats)
    if re.fullmatch("mid_[nt][nt]", base) and checked != 4:
        raise RuntimeError(f"{obj}: {checked} kernels with asm-held accumulators, not 4")
    return checked


def build(verbose: bool = False) -> str:
    """Compile the library (always recompiles). Returns its path."""
    sources = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    with tempfile.TemporaryDirectory(prefix="scalify_build_") as tmp:
        def compile_one(src: str) -> str:
            obj = os.path.join(tmp, os.path.basename(src) + ".o")
            cmd = [_hipcc(), *HIPCC_FLAGS, "-c", src, "-o", obj]
            r = subprocess.run(cmd, capture_output=True, text=True)
            if r.returncode != 0:
                raise RuntimeError(f"hipcc failed for {src}:\n{r.stderr}")
            if verbose and r.stderr.strip():
                print(r.stderr)
            if os.path.basename(src).startswith(("gemm_", "mid_", "wave_")):
                check_code(obj, tmp)
            return obj

        workers = min(len(sources), max(1, os.cpu_count() or 1), 8)
        with cf.ThreadPoolExecutor(workers) as ex:
            objs = list(ex.map(compile_one, sources))
        tmp_lib = LIB + ".tmp"
        cmd = [_hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp_lib, *objs]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"link failed:\n{r.stderr}")
        os.replace(tmp_lib, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
