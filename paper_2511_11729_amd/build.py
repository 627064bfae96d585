"""Builds libharli.so (HIP, gfx950) in-tree with hipcc.

    python -m paper_2511_11729_amd.build

The library is a plain C-ABI shared object (no torch types); `binding.py` loads
it with ctypes.
"""
from __future__ import annotations

import os
import re
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libharli.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
COMMON = ["-O3", "-std=c++17", "-fPIC", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "-Wall", "-Wno-unused-function"]
# packed-fp32 VALU forms are switched off: -O3 would otherwise form v_pk_*_f32 from scalar float code
HIPFLAGS = ["--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def sources():
    out = []
    for f in sorted(os.listdir(CSRC)):
        if f.endswith(".hip") or f.endswith(".cpp"):
            out.append(os.path.join(CSRC, f))
    return out


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, os.path.basename(src) + ".o")
    cmd = [HIPCC] + COMMON + (HIPFLAGS if src.endswith(".hip") else []) + ["-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    msgs = "\n".join(l for l in (r.stdout + r.stderr).splitlines()
                     if "packed-fp32-ops" not in l and "is not a recognized feature" not in l)
    if r.returncode != 0:
        raise RuntimeError("compile failed: %s\n%s" % (" ".join(cmd), msgs))
    if msgs.strip():
        print(msgs, file=sys.stderr)
    return obj


def device_listing(obj: str, kernels: str) -> dict:
    """(address, instruction) of the gfx950 code in an object built here, by symbol, for the symbols that hold `kernels`."""
    llvm = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(HIPCC))), "lib", "llvm", "bin")
    if not os.path.exists(llvm):
        llvm = "/opt/rocm/llvm/bin"
    out = {}
    with tempfile.TemporaryDirectory() as d:
        fat, code = os.path.join(d, "fat"), os.path.join(d, "code")

        def tool(name, *args):
            r = subprocess.run([os.path.join(llvm, name), *args], capture_output=True, text=True)
            if r.returncode != 0:
                raise RuntimeError("%s failed on %s:\n%s" % (name, obj, r.stderr))
            return r.stdout

        tool("llvm-objcopy", "--dump-section=.hip_fatbin=" + fat, obj, os.path.join(d, "copy.o"))
        tool("clang-offload-bundler", "--unbundle", "--type=o", "--input=" + fat, "--output=" + code,
             "--targets=hipv4-amdgcn-amd-amdhsa--gfx950")
        name = None
        for line in tool("llvm-objdump", "-d", "--no-show-raw-insn", code).splitlines():
            m = re.match(r"[0-9a-f]+ <(\w+)>:", line)
            if m:
                name = m.group(1) if kernels in m.group(1) else None
            elif name and line.startswith("\t") and "//" in line:   # (no address: zeros between two kernels)
                ins, _, where = line.partition("//")
                out.setdefault(name, []).append((int(where.split(":")[0], 16), ins.strip()))
    return out


_ACC = re.compile(r"\ba(?:\d+|\[[0-9a-fx:]+\])")
_VEC = re.compile(r"\bv(?:(\d+)|\[(\d+):(\d+)\])")


def _vector_registers(operand: str) -> set:
    out = set()
    for one, lo, hi in _VEC.findall(operand):
        out |= {int(one)} if one else set(range(int(lo), int(hi) + 1))
    return out


def _split(ins: str):
    op = ins.split(None, 1)[0]
    return op, [a.strip() for a in ins[len(op):].split(",")]


def _vector_writes(ins: str) -> set:
    """Vector registers a vector instruction writes (products and accumulator moves left out)."""
    op, args = _split(ins)
    if not op.startswith("v_") or op.startswith(("v_mfma_", "v_accvgpr_write")):
        return set()
    return _vector_registers(ins if op.startswith(("v_permlane", "v_swap")) else args[0])   # those write both operands


def check_named_accumulators(name: str, code: list) -> None:
    """Raises unless a kernel whose accumulator registers are named in inline assembly is safe from the compiler, which knows
    neither the accumulators nor that the assembly holds matrix instructions: accumulator registers in nothing but products
    (a sum onto itself), zeros and reads, no spill, and no vector instruction that writes a product's operand in the two
    slots before it, along either way of a branch (the wait states the compiler fills in only for products it knows)."""
    at = {address: i for i, (address, _) in enumerate(code)}
    before = [set() for _ in code]                  # instructions that may run right before this one
    for i, (address, ins) in enumerate(code):
        op, args = _split(ins)
        if op not in ("s_branch", "s_endpgm", "s_setpc_b64") and i + 1 < len(code):
            before[i + 1].add(i)
        if op.startswith(("s_branch", "s_cbranch")):
            offset = int(args[0], 0)
            before[at[address + 4 + 4 * (offset - 65536 if offset > 32767 else offset)]].add(i)
    for i, (address, ins) in enumerate(code):
        op, args = _split(ins)
        product = op.startswith("v_mfma_")
        if op.startswith(("scratch_", "v_accvgpr_mov")):
            raise RuntimeError("%s: %s: a spill or an accumulator copy" % (name, ins))
        acc = _ACC.findall(ins)
        if acc and not (product and len(acc) == 2 and acc[0] == acc[1] == args[0] or op.startswith("v_accvgpr_write") and args[1] == "0"
                        or op.startswith("v_accvgpr_read")):
            raise RuntimeError("%s: %s: an accumulator register in an instruction the source does not write" % (name, ins))
        if product:
            reads = _vector_registers(args[1]) | _vector_registers(args[2])
            for j in before[i]:
                near = {j} if _split(code[j][1])[0] == "s_nop" and code[j][1].split()[1] != "0" else {j} | before[j]
                for k in near:
                    if reads & _vector_writes(code[k][1]):
                        raise RuntimeError("%s: %s: an operand is written by %s, less than two slots before" % (name, ins, code[k][1]))


def _check(obj: str) -> None:
    if os.path.basename(obj).startswith("gemm2_rows"):
        kernels = device_listing(obj, "k_gemm2I")
        if not kernels:
            raise RuntimeError("%s holds no weight GEMM" % obj)
        for name, code in kernels.items():
            check_named_accumulators(name, code)


def build_lib(verbose: bool = True) -> str:
    os.makedirs(OBJ, exist_ok=True)
    srcs = sources()
    with ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(_compile, srcs))
        list(ex.map(_check, objs))
    cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", LIB] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout + r.stderr)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build_lib()
