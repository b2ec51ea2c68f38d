"""Build-time guard of the kernel that holds dK/dV and dQ: no early read of an asm MFMA's result, no copy to LDS that reads
a scalar too early, no spill inside its loops, and registers for two wavefronts per SIMD."""
import re

import pytest

from test_build_guards import kernel_instructions, kernel_metadata
from test_build_guards_eight_waves import backward_asm, early_reads_of_asm_mfma_results, late_scalars_of_copies


@pytest.mark.parametrize("shared", [0, 1])
@pytest.mark.parametrize("d", [64, 128])
def test_the_kernel_with_both(d, shared):
    text = backward_asm()
    name = next(k for k in kernel_metadata(text) if re.search(r"bwd_both_kernelILi%dELi%dELb%d" % (d, d, shared), k))
    ins = kernel_instructions(text, name)
    assert early_reads_of_asm_mfma_results(ins) == []
    assert late_scalars_of_copies(ins) == []
    mfma = [i for i, l in enumerate(ins) if l.startswith("v_mfma")]
    # one reload between the two bodies is allowed; none within 64 instructions of a matrix instruction
    near = [i for i, l in enumerate(ins) if l.startswith("scratch_") and any(abs(i - m) < 64 for m in mfma)]
    assert near == []
    regs = int(re.search(r"\.name:\s+%s\n(?:.*\n)*?\s+\.vgpr_count:\s+(\d+)" % name, text).group(1))
    assert regs <= 256


def test_the_kernel_with_both_at_head_size_192():
    text = backward_asm()
    name = next(k for k in kernel_metadata(text) if "bwd_both4_kernelILi192E" in k)
    ins = kernel_instructions(text, name)
    assert early_reads_of_asm_mfma_results(ins) == [] and late_scalars_of_copies(ins) == []
    assert not any(l.startswith("scratch_") for l in ins)
    assert int(re.search(r"\.name:\s+%s\n(?:.*\n)*?\s+\.vgpr_count:\s+(\d+)" % name, text).group(1)) <= 512
