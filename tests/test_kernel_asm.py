"""Static checks on the device code of the four-wave GEMM kernel (no GPU needed: hipcc cross-compiles).

Its K loop keeps 256 accumulators in AGPRs through inline-assembly MFMAs with one wave per SIMD; two things the
compiler may do when register allocation gets tight would ruin it without failing any numerical test outright:
spilling inside the loop (the loop then waits on scratch memory), and moving accumulators with v_accvgpr_write /
v_accvgpr_mov right in front of an inline MFMA (whose read-after-write hazard the compiler does not pad, since it
cannot see the instruction).  Both are looked for in the assembly of every instantiation."""
import re
import shutil
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parent.parent
CSRC = ROOT / "paper_2209_13258_amd" / "csrc"


@pytest.fixture(scope="module")
def gemm_asm(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not Path(hipcc).exists():
        pytest.skip("hipcc not found")
    out = tmp_path_factory.mktemp("asm") / "osdp_gemm.s"
    cmd = [hipcc, "-O3", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           f"-I{ROOT / 'include'}", f"-I{CSRC}", "-S", "--cuda-device-only", str(CSRC / "osdp_gemm.hip"), "-o", str(out)]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    return out.read_text().split("\n")


def _kernels(lines, kernel="gemm_w4_kernel"):
    """{mangled name: list of instruction lines} for the instantiations of one kernel template."""
    kernels, cur = {}, None
    for line in lines:
        m = re.match(r"^(_ZN4osdp\S*" + kernel + r"I\S*):", line)
        if m:
            cur = m.group(1)
            kernels[cur] = []
            continue
        if re.match(r"^\S+:", line) and not line.startswith(".L"):   # another function starts
            cur = None
        t = line.strip()
        if cur and t and not t.startswith((";", ".")):
            kernels[cur].append(t)
    return kernels


def _vgprs(operand):
    """The VGPR numbers an operand like v7 or v[8:11] names (empty for anything else)."""
    m = re.fullmatch(r"v(\d+)", operand)
    if m:
        return {int(m.group(1))}
    m = re.fullmatch(r"v\[(\d+):(\d+)\]", operand)
    return set(range(int(m.group(1)), int(m.group(2)) + 1)) if m else set()


def _assert_no_valu_write_in_front_of_its_mfma(name, ins, mfma):
    """An MFMA may not read a register in the two cycles after a VALU instruction wrote it; the compiler pads none
    for an MFMA it cannot see."""
    for i in mfma:
        ops = [o.strip() for o in ins[i].split(None, 1)[1].split(",")]
        srcs = _vgprs(ops[1]) | _vgprs(ops[2])
        for t in ins[max(0, i - 2):i]:
            if t.startswith("v_") and not t.startswith("v_mfma"):
                dst = t.split(None, 1)[1].split(",")[0].strip()
                assert not (_vgprs(dst) & srcs), f"{name}: '{t}' writes a source of the MFMA that follows it"


def test_four_wave_kernels_keep_their_k_loop_free_of_scratch_and_accumulator_moves(gemm_asm):
    kernels = _kernels(gemm_asm)
    assert len(kernels) >= 12, "the four-wave kernel's instantiations were not found in the assembly"
    for name, ins in kernels.items():
        mfma = [i for i, t in enumerate(ins) if t.startswith("v_mfma")]
        assert len(mfma) == 128, f"{name}: expected one K block of 128 MFMAs, found {len(mfma)} (the loop body was duplicated?)"
        body = ins[mfma[0]:mfma[-1] + 1]
        assert not [t for t in body if t.startswith("scratch_")], f"{name}: scratch traffic inside the K loop"
        for i in mfma:
            near = ins[max(0, i - 3):i]
            assert not [t for t in near if t.startswith(("v_accvgpr_write", "v_accvgpr_mov"))], \
                f"{name}: an accumulator register is written right in front of an inline MFMA"
        _assert_no_valu_write_in_front_of_its_mfma(name, ins, mfma)


def test_persistent_four_wave_kernels_use_no_scratch_and_respect_the_mfma_hazards(gemm_asm):
    """The persistent form runs its epilogue and the start of the next tile inside the loop over K blocks, where the
    compiler has no register to spare: any spill there, any accumulator moved by the compiler, or a source
    register of an inline MFMA written by a VALU instruction just before it (two wait states are needed, and the
    compiler pads none for an instruction it cannot see) is a defect."""
    kernels = _kernels(gemm_asm, "gemm_w4p_kernel")
    assert len(kernels) >= 10, "the persistent kernel's instantiations were not found in the assembly"
    for name, ins in kernels.items():
        assert not [t for t in ins if t.startswith("scratch_")], f"{name}: scratch traffic"
        mfma = [i for i, t in enumerate(ins) if t.startswith("v_mfma")]
        # one K block of 128, plus 64 that clear the accumulators before the first tile and 64 between tiles
        # (instantiations that start from a stored partial sum load it instead)
        assert len(mfma) in (128, 256), f"{name}: {len(mfma)} MFMAs"
        for i in mfma:
            near = ins[max(0, i - 3):i]
            assert not [t for t in near if t.startswith(("v_accvgpr_write", "v_accvgpr_mov"))], \
                f"{name}: an accumulator register is written right in front of an inline MFMA"
        _assert_no_valu_write_in_front_of_its_mfma(name, ins, mfma)


def test_four_wave_kernels_of_smaller_tiles_keep_the_same_rules(gemm_asm):
    """32 * MB x 32 * NB tiles: one K block of 2 * MB * NB MFMAs (the persistent form clears as many again)."""
    for kernel, counts in (("gemm_w4_small_kernel", (1,)), ("gemm_w4p_small_kernel", (1, 2))):
        kernels = _kernels(gemm_asm, kernel)
        assert len(kernels) >= 10, f"the instantiations of {kernel} were not found in the assembly"
        for name, ins in kernels.items():
            mb, nb = map(int, re.search(kernel + r"ILi(\d+)ELi(\d+)E", name).groups())
            mfma = [i for i, t in enumerate(ins) if t.startswith("v_mfma")]
            assert len(mfma) in [2 * mb * nb * c for c in counts], f"{name}: {len(mfma)} MFMAs"
            assert not [t for t in ins[mfma[0]:mfma[-1] + 1] if t.startswith("scratch_")], f"{name}: scratch traffic inside the K loop"
            for i in mfma:
                assert not [t for t in ins[max(0, i - 3):i] if t.startswith(("v_accvgpr_write", "v_accvgpr_mov"))], \
                    f"{name}: an accumulator register is written right in front of an inline MFMA"
            _assert_no_valu_write_in_front_of_its_mfma(name, ins, mfma)


@pytest.mark.parametrize("kernel,least", [("gemm_w4_128_kernel", 20), ("gemm_w4_160_kernel", 4)])
def test_four_wave_kernels_of_lone_tiles_keep_the_same_rules(gemm_asm, kernel, least):
    """32 * MB x 32 * NB tiles: one K block of 2 * MB * NB MFMAs, and every load of a block has its place."""
    kernels = _kernels(gemm_asm, kernel)
    assert len(kernels) >= least, "the instantiations were not found in the assembly"
    for name, ins in kernels.items():
        mb, nb = (4, 4) if "128" in kernel else (int(re.search(kernel + r"ILi(\d+)E", name).group(1)), 5)
        mfma = [i for i, t in enumerate(ins) if t.startswith("v_mfma")]
        assert len(mfma) == 2 * mb * nb, f"{name}: {len(mfma)} MFMAs"
        loads = [t for t in ins[mfma[0]:] if t.startswith("buffer_load") and t.endswith(" lds")]
        assert len(loads) == mb + nb, f"{name}: {len(loads)} loads in a K block"
        assert not [t for t in ins if t.startswith("scratch_")], f"{name}: scratch traffic"
        for i in mfma:
            assert not [t for t in ins[max(0, i - 3):i] if t.startswith(("v_accvgpr_write", "v_accvgpr_mov"))], \
                f"{name}: an accumulator register is written right in front of an inline MFMA"
        _assert_no_valu_write_in_front_of_its_mfma(name, ins, mfma)


def _inline_mfmas(lines, kernel):
    """{mangled name: (instructions, indices of the MFMAs that stand in inline assembly)}: the compiler marks what it did
    not write itself, and pads the hazards of its own MFMAs."""
    out, cur, inline = {}, None, False
    for line in lines:
        m = re.match(r"^(_ZN4osdp\S*" + kernel + r"I\S*):", line)
        if m:
            cur = out.setdefault(m.group(1), ([], []))
            continue
        if re.match(r"^\S+:", line) and not line.startswith(".L"):   # another function starts
            cur = None
        t = line.strip()
        if t.startswith((";;#ASMSTART", ";;#ASMEND")):
            inline = "START" in t
        elif cur and t and not t.startswith((";", ".")):
            if inline and t.startswith("v_mfma"):
                cur[1].append(len(cur[0]))
            cur[0].append(t)
    return out


def _accumulators(operand):
    """The AGPR numbers an operand like a7 or a[8:11] names (empty for anything else)."""
    return _vgprs("v" + operand[1:]) if operand.startswith("a") else set()


def _accumulator_writes_near(ins, mfma):
    """(write, MFMA) pairs where one of the three instructions in front of an inline MFMA writes a register that it adds to."""
    pairs = []
    for i in mfma:
        acc = _accumulators(ins[i].split(None, 1)[1].split(",")[0].strip())
        for t in ins[max(0, i - 3):i]:
            if t.startswith(("v_accvgpr_write", "v_accvgpr_mov")) and _accumulators(t.split(None, 1)[1].split(",")[0].strip()) & acc:
                pairs.append((t, ins[i]))
    return pairs


def test_the_backward_of_few_tokens_keeps_the_same_rules_for_its_dw_tiles(gemm_asm):
    """few_token_backward_kernel holds the loop of a 128 x 128 tile, whose 32 MFMAs the compiler cannot see, beside dX's, which
    it schedules and pads by itself and which share the register file: the rules are for the inline ones."""
    kernels = _inline_mfmas(gemm_asm, "few_token_backward_kernel")
    assert len(kernels) == 3, "the instantiations were not found in the assembly"
    for name, (ins, mfma) in kernels.items():
        assert len(mfma) == 32, f"{name}: {len(mfma)} inline MFMAs"
        assert len([t for t in ins if t.startswith("v_mfma")]) > 32, f"{name}: dX's own MFMAs were not found"
        assert not [t for t in ins if t.startswith("scratch_")], f"{name}: scratch traffic"
        assert not _accumulator_writes_near(ins, mfma), f"{name}: an accumulator register is written right in front of an inline MFMA"
        _assert_no_valu_write_in_front_of_its_mfma(name, ins, mfma)


def test_the_rules_for_inline_mfmas_find_a_planted_write():
    """The two searches on a few lines of assembly: a write of an accumulator, and of a source, that the MFMA reads; the same
    writes before an MFMA of the compiler's own, or of other registers, are none of theirs."""
    head, tail = "_ZN4osdp1_25few_token_backward_kernelILi16EEEv:", "\ts_endpgm"
    mfma = "\tv_mfma_f32_16x16x32_bf16 a[8:11], v[4:7], v[0:3], a[8:11]"
    inline = ["\t;;#ASMSTART", mfma, "\t;;#ASMEND"]

    def look(before, body=inline):
        (name, (ins, found)), = _inline_mfmas([head] + before + body + [tail], "few_token_backward_kernel").items()
        return name, ins, found

    for write, hit in (("v_accvgpr_write_b32 a9, v20", True), ("v_accvgpr_write_b32 a12, v20", False), ("v_accvgpr_mov_b32 a[10:10], a1", True)):
        name, ins, found = look(["\t" + write, "\ts_nop 1"])
        assert bool(_accumulator_writes_near(ins, found)) == hit, write
        name, ins, found = look(["\t" + write], [mfma])
        assert not found
    for write, hit in (("v_add_u32_e32 v5, 1, v9", True), ("v_add_u32_e32 v8, 1, v9", False)):
        name, ins, found = look(["\t" + write])
        if hit:
            with pytest.raises(AssertionError):
                _assert_no_valu_write_in_front_of_its_mfma(name, ins, found)
        else:
            _assert_no_valu_write_in_front_of_its_mfma(name, ins, found)
