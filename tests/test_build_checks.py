"""CPU checks of the compiled dK/dV kernels (head_dim 128), which update their accumulators in place by inline assembly: the
compiler does not know how long such an accumulator takes to be written, so nothing else may touch its registers in between."""
import os
import re
import subprocess

import pytest

from paper_2503_02356_amd import build

REPORT = """a.hip:1:1: remark: Function Name: _ZN2cf16mfma_dkv_kernelILi128ELb0EEEv [-Rpass-analysis=kernel-resource-usage]
a.hip:1:1: remark:     ScratchSize [bytes/lane]: {scratch} [-Rpass-analysis=kernel-resource-usage]
a.hip:1:1: remark:     SGPRs Spill: 3 [-Rpass-analysis=kernel-resource-usage]
a.hip:1:1: remark:     VGPRs Spill: {spill} [-Rpass-analysis=kernel-resource-usage]
a.hip:1:1: remark: Function Name: _ZN2cf14mfma_dq_kernelILi128EEEv [-Rpass-analysis=kernel-resource-usage]
a.hip:1:1: remark:     VGPRs Spill: 9 [-Rpass-analysis=kernel-resource-usage]
"""


def test_a_spilled_accumulator_fails_the_build():
    assert build.spilled_accumulators(REPORT.format(scratch=0, spill=0)) == []
    assert len(build.spilled_accumulators(REPORT.format(scratch=8, spill=2))) == 2


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs hipcc")
def test_no_fp32_kernel_spills():
    report = subprocess.run([build.HIPCC] + build.HIP_FLAGS + [build.RESOURCE_REPORT, "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC,
                             "--cuda-device-only", "-c", os.path.join(build.CSRC, "attn_fp32.hip"), "-o", os.devnull], check=True,
                            stderr=subprocess.PIPE, text=True).stderr
    assert len(re.findall(r"Function Name: \S*f32_bwd_batch_kernel", report)) == 2
    assert build.spilled_operands(report) == []
    assert build.spilled_operands(REPORT.format(scratch=8, spill=2))      # (another kernel's spill is seen)


def registers(operand):
    m = re.fullmatch(r"v\[(\d+):(\d+)\]|v(\d+)", operand)
    return set() if m is None else {int(m[3])} if m[3] else set(range(int(m[1]), int(m[2]) + 1))


def operands(line):
    return re.split(r",?\s+", line.split(";")[0].strip())[1:]


def accumulator_faults(text):
    """Instructions of a kernel that use a register of an in-place accumulator between the first and the last in-place MFMA."""
    lines = [l.strip() for l in text.splitlines()]
    lines = [l for l in lines if l and not l.startswith((";", ".", "//")) and not l.endswith(":")]
    mfma = [i for i, l in enumerate(lines) if l.startswith("v_mfma_f32_32x32x16_bf16") and lines[i - 1] == "s_nop 1"
            and operands(l)[0] == operands(l)[3]]
    accumulators = set().union(*(registers(operands(lines[i])[0]) for i in mfma))
    faults = [l for i, l in enumerate(lines) if mfma[0] <= i <= mfma[-1] and i not in mfma
              and any(registers(o) & accumulators for o in operands(l))]
    return len(mfma), len(accumulators), faults


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs hipcc")
def test_nothing_else_touches_an_accumulator_in_the_loop(tmp_path):
    out = str(tmp_path / "bwd.s")
    subprocess.run([build.HIPCC] + build.HIP_FLAGS + ["-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, "--cuda-device-only",
                   "-S", os.path.join(build.CSRC, "attn_mfma_bwd.hip"), "-o", out], check=True, stderr=subprocess.DEVNULL)
    text = open(out).read()
    kernels = re.findall(r"^(\S*mfma_dkv\S*ILi128E\S*):.*?\n(.*?)^\.Lfunc_end", text, re.M | re.S)
    assert len(kernels) == 4
    for name, body in kernels:
        n, regs, faults = accumulator_faults(body)
        assert n > 0 and regs == 128 and faults == [], (name, n, regs, faults[:5])
        # (the check sees a use that is planted between two of them)
        last = list(re.finditer(r"s_nop 1\n\s*(v_mfma_f32_32x32x16_bf16 .*)\n", body))[-1]
        planted = body[:last.start()] + f"v_mov_b32_e32 v0, v{min(registers(operands(last[1])[0]))}\n\t" + body[last.start():]
        assert accumulator_faults(planted)[2]


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs hipcc")
def test_products_of_dq_alternate(tmp_path):
    """S and dP are one chain of 32x32x16 MFMAs each: no two in a row add to the same accumulator, which would have to wait."""
    out = str(tmp_path / "bwd.s")
    subprocess.run([build.HIPCC] + build.HIP_FLAGS + ["-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, "--cuda-device-only",
                   "-S", os.path.join(build.CSRC, "attn_mfma_bwd.hip"), "-o", out], check=True, stderr=subprocess.DEVNULL)
    kernels = re.findall(r"^(\S*mfma_dq_\S+):.*?\n(.*?)^\.Lfunc_end", open(out).read(), re.M | re.S)
    assert len(kernels) >= 4
    for name, body in kernels:
        mfma = [operands(l.strip())[0] for l in body.splitlines() if l.strip().startswith("v_mfma")]
        assert len(mfma) > 100 and all(a != b for a, b in zip(mfma, mfma[1:])), name


def lane_faults(text):
    """Inline assembly blocks (between the compiler's marks) in which a vector instruction writes a scalar register, whose later uses the
    compiler then does not hold back, and lane reads right behind a block that wrote their register, for which it puts no wait state."""
    lines = [l.strip() for l in text.splitlines()]
    lines = [l for l in lines if l and (l.startswith(";;#ASM") or not l.startswith((";", ".", "//")) and not l.endswith(":"))]
    faults, inside, last = [], False, ""
    for line in lines:
        if line.startswith(";;#ASM"):
            inside = line == ";;#ASMSTART"
        elif inside:
            if re.match(r"v_\S+\s+(s\d|s\[|vcc|exec)", line):
                faults.append(line)
            last = line
        else:
            if re.match(r"v_read(first)?lane", line) and last.startswith("v_") and registers(operands(line)[1]) & registers(operands(last)[0]):
                faults.append(line)
            last = ""
    return faults


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs hipcc")
def test_lane_reads_are_the_compilers(tmp_path):
    """A lane read needs a wait state behind the instruction that wrote its register, and what uses its scalar result up to five behind it
    (a memory access); the compiler sees to both for its own instructions, not for those of inline assembly."""
    for name in build.HIP_SOURCES:
        out = str(tmp_path / (name + ".s"))
        subprocess.run([build.HIPCC] + build.HIP_FLAGS + ["-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, "--cuda-device-only",
                       "-S", os.path.join(build.CSRC, name), "-o", out], check=True, stderr=subprocess.DEVNULL)
        text = open(out).read()
        assert lane_faults(text) == [], name
        # (the check sees both kinds where they are planted)
        planted = text + ";;#ASMSTART\n\tv_readfirstlane_b32 s7, v2\n\t;;#ASMEND\n;;#ASMSTART\n\tv_mov_b32_e32 v3, v4\n\t;;#ASMEND\n\tv_readlane_b32 s8, v3, 1\n"
        assert len(lane_faults(planted)) == 2
    assert "#ASMSTART" in text
