"""The finetune unit's weight GEMM names its accumulator registers by hand (inline assembly): the compiled kernels may touch
accumulator registers only in the instructions the source writes.  A copy or a spill the compiler put among them would
change a sum without any error, so the built object is read back (no GPU)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2511_11729_amd.build import check_named_accumulators, device_listing

HERE = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
OBJS = [os.path.join(HERE, "paper_2511_11729_amd", "_build", "gemm2_rows%d.hip.o" % r) for r in (128, 160, 192, 224, 256)]
LLVM = "/opt/rocm/llvm/bin"
ACC = re.compile(r"\ba(?:\d+|\[[0-9a-fx:]+\])")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not all(os.path.exists(o) for o in OBJS) or not shutil.which(os.path.join(LLVM, "llvm-objdump")):
        pytest.skip("needs the built objects and the ROCm LLVM tools")
    d = tmp_path_factory.mktemp("isa")
    out = {}
    for obj in OBJS:
        fat, code = str(d / "fat"), str(d / "code")
        subprocess.run([LLVM + "/llvm-objcopy", "--dump-section=.hip_fatbin=" + fat, obj, str(d / "copy.o")], check=True)
        subprocess.run([LLVM + "/clang-offload-bundler", "--unbundle", "--type=o", "--input=" + fat, "--output=" + code,
                        "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"], check=True)
        text = subprocess.run([LLVM + "/llvm-objdump", "-d", "--no-show-raw-insn", code], check=True, capture_output=True, text=True).stdout
        name = None
        for line in text.splitlines():
            m = re.match(r"[0-9a-f]+ <(\w+)>:", line)
            if m:
                name = m.group(1)
            elif name and "k_gemm2I" in name and line.startswith("\t"):
                out.setdefault(name, []).append(line.split("//")[0].strip())
    return out


def test_accumulators_are_touched_by_the_written_instructions_alone(kernels):
    assert len(kernels) == 5 * 5 + 2 * 4
    for name, code in kernels.items():
        rt = int(re.search(r"k_gemm2ILi(\d+)E", name).group(1))
        n = {"v_mfma": 0, "zero": 0, "read": 0}
        for ins in code:
            assert not ins.startswith(("scratch_", "v_accvgpr_mov")), (name, ins)
            if not ACC.search(ins):
                continue
            if ins.startswith("v_mfma_f32_16x16x32_"):
                regs = ACC.findall(ins)
                assert len(regs) == 2 and regs[0] == regs[1], (name, ins)   # the sum alone, onto itself
                n["v_mfma"] += 1
            elif ins.startswith("v_accvgpr_write_b32"):
                assert ins.endswith(", 0"), (name, ins)
                n["zero"] += 1
            else:
                assert ins.startswith("v_accvgpr_read_b32"), (name, ins)
                n["read"] += 1
        # two stages a pass of the loop; zeros before the loop and where a tile has no stage; epilogue and partial tiles read
        assert n == {"v_mfma": 2 * 8 * rt, "zero": 2 * 32 * rt, "read": 2 * 32 * rt}, (name, n)


# ---- the same reading refuses a build (paper_2511_11729_amd/build.py) --------------------------------------------------
def listing(*lines):
    return [(4 * i, ins) for i, ins in enumerate(lines)]


MM = "v_mfma_f32_16x16x32_f16 a[0:3], v[18:21], v[62:65], a[0:3]"


@pytest.mark.parametrize("lines", [
    ("v_mov_b32_e32 v18, v2", MM),                                            # right before the product
    ("v_mov_b32_e32 v64, v2", "s_add_i32 s2, s31, s52", MM),                  # one slot between
    ("v_mov_b32_e32 v64, v2", "s_nop 0", MM),
    ("v_permlane16_swap_b32_e32 v1, v20", "s_nop 0", MM),                     # the second operand is written too
    (MM, "v_add_u32_e32 v21, s64, v1", "s_cbranch_scc1 65533", "s_endpgm"),   # along a loop's back edge
    ("v_mfma_f32_16x16x32_f16 a[0:3], v[18:21], v[62:65], a[4:7]",),          # a sum onto another
    ("v_mfma_f32_16x16x32_f16 v[0:3], v[18:21], v[62:65], a[0:3]",),
    ("v_accvgpr_write_b32 a7, v3",), ("v_accvgpr_mov_b32 a7, a8",), ("global_store_dwordx4 v0, a[0:3], s[2:3]",),
    ("scratch_store_dword off, v3, s32",)])
def test_a_planted_fault_is_refused(lines):
    with pytest.raises(RuntimeError):
        check_named_accumulators("planted", listing(*lines))


@pytest.mark.parametrize("lines", [
    ("v_mov_b32_e32 v18, v2", "s_nop 0", "s_nop 0", MM), ("v_mov_b32_e32 v18, v2", "s_nop 1", MM), ("v_mov_b32_e32 v22, v2", MM),
    ("v_accvgpr_write_b32 a3, 0", MM, "v_accvgpr_read_b32 v18, a3"),
    (MM, "v_add_u32_e32 v21, s64, v1", "s_nop 0", "s_cbranch_scc1 65532", "s_endpgm"),
    (MM, "s_cbranch_scc1 2", "v_mov_b32_e32 v18, v2", "s_nop 1", MM)])       # either way of a branch
def test_what_is_sound_passes(lines):
    check_named_accumulators("sound", listing(*lines))


def test_the_built_kernels_pass():
    if not all(os.path.exists(o) for o in OBJS):
        pytest.skip("needs the built objects")
    n = 0
    for obj in OBJS:
        for name, code in device_listing(obj, "k_gemm2I").items():
            check_named_accumulators(name, code)
            n += 1
    assert n == 5 * 5 + 2 * 4
