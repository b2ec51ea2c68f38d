"""Build-time guards of the dK/dV kernel with eight wavefronts, as for the other kernels with asm MFMAs, and of the
copies through buffer descriptors."""
import re

import pytest

from test_build_guards import backward_asm, early_reads_of_asm_mfma_results, kernel_instructions, kernel_metadata


def registers(text):
    out = {int(x) for x in re.findall(r"\bs(\d+)\b", text)}
    for a, b in re.findall(r"\bs\[(\d+):(\d+)\]", text):
        out |= set(range(int(a), int(b) + 1))
    return out


def late_scalars_of_copies(ins, need=5):
    """Copies to LDS that read a scalar register fewer than `need` wait states after a vector instruction wrote it
    (a spilled scalar comes back that way); the compiler does not see that the asm is a memory instruction."""
    found = []
    for i, l in enumerate(ins):
        if not re.match(r"(buffer|global)_load\w*\s.*\blds\b|global_load_lds", l):
            continue
        reads, states = registers(l.split(None, 1)[1]), 0
        for p in reversed(ins[max(0, i - need):i]):
            if states >= need:
                break
            if re.match(r"v_(readlane|readfirstlane|cmp)", p) and registers(p.split(None, 1)[1].split(",")[0]) & reads:
                found.append((p, l, states))
                break
            states += int(p.split()[1]) + 1 if p.startswith("s_nop") else 1
    return found


def test_the_scan_of_scalars_sees_a_planted_one():
    late = ["v_readlane_b32 s3, v9, 1", "s_add_u32 m0, s4, 0", "s_nop 0", "buffer_load_dwordx4 v1, s[0:3], 0 offen lds"]
    assert len(late_scalars_of_copies(late)) == 1
    assert late_scalars_of_copies(late[:1] + ["s_nop 4"] + late[1:]) == []
    assert late_scalars_of_copies(["v_readlane_b32 s4, v9, 1"] + late[1:]) == []


@pytest.mark.parametrize("d", [64, 128])
def test_the_eight_wave_kernel(d):
    text = backward_asm()
    meta = kernel_metadata(text)
    name = next(k for k in meta if "bwd_dkdv8_kernelILi%dE" % d in k)
    ins = kernel_instructions(text, name)
    assert any(re.match(r"v_mfma_f32_32x32x16_bf16 v\[", l) for l in ins)
    assert early_reads_of_asm_mfma_results(ins) == []
    assert late_scalars_of_copies(ins) == []
    mfma = [i for i, l in enumerate(ins) if l.startswith("v_mfma")]
    scratch = [i for i, l in enumerate(ins) if l.startswith("scratch_")]
    assert all(i < mfma[0] or i > mfma[-1] + 64 for i in scratch), (scratch, mfma[0], mfma[-1])
    assert not any("v_accvgpr_mov" in l for l in ins)
    regs = int(re.search(r"\.name:\s+%s\n(?:.*\n)*?\s+\.vgpr_count:\s+(\d+)" % name, text).group(1))
    assert regs <= 256  # two wavefronts per SIMD
    # What is parked in scratch is written and read again by every item, in front of and behind its steps: no more of it
    # than there is (vector registers, scalar registers, bytes a lane).
    block = next(b for b in re.findall(r"  - \.agpr_count:.*?\.wavefront_size:", text, re.S) if name in b)
    spills = [int(re.search(r"\.%s:\s+(\d+)" % k, block).group(1))
              for k in ("vgpr_spill_count", "sgpr_spill_count", "private_segment_fixed_size")]
    assert all(a <= b for a, b in zip(spills, {64: (0, 78, 0), 128: (17, 85, 80)}[d])), spills
