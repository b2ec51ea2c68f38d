"""Build-time guard: in kernels that use the inline-asm MFMA form no register spill or reload may sit among
the MFMAs (a spill copy next to an asm MFMA would escape the compiler's hazard handling: the compiler does
not see what the asm writes and when).  A value parked in scratch once per work item, in the item's
prologue far ahead of the first MFMA, is harmless and allowed.  Nor may any vector instruction touch the result
registers of an asm MFMA before the result exists: the compiler inserts such a read when it joins the score
registers of two code paths by copies (it has happened: wrong dK on every pack of short samples), and no
run-time check tells it from rounding noise on long ones."""
import os
import re
import subprocess
import tempfile

import pytest

from paper_2503_07680_amd import build as B


def kernel_metadata(asm_text):
    out = {}
    for m in re.finditer(r"\.name:\s+(\S+)\n(?:.*\n)*?\s+\.vgpr_spill_count:\s+(\d+)", asm_text):
        out[m.group(1)] = int(m.group(2))
    return out


_ASM_CACHE = {}


def device_asm(source, flags=()):
    key = (source, *flags)
    if key not in _ASM_CACHE:
        with tempfile.TemporaryDirectory() as tmp:
            out = os.path.join(tmp, "out.s")
            cmd = [B._hipcc()] + B.HIP_FLAGS + [*flags, "-S", "--cuda-device-only", os.path.join(B.CSRC, source), "-o", out]
            subprocess.run(cmd, check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
            _ASM_CACHE[key] = open(out).read()
    return _ASM_CACHE[key]


def backward_asm():
    return device_asm("bwd.hip")


def kernel_instructions(text, name):
    body = text[text.index("\n" + name + ":"):]
    body = body[:body.index(".end_amdhsa_kernel")]
    return [l.strip() for l in body.splitlines()
            if l.startswith("\t") and l.strip() and not l.strip().startswith((";", "."))]


def early_reads_of_asm_mfma_results(ins, need=18):
    """Instructions that name a register of an asm MFMA's destination tuple (the asm form writes vector
    registers, v[a:b]; the builtin form writes accumulation registers here) fewer than `need` wait states
    behind that MFMA.  Another MFMA ends the window (a chain on the same accumulator is interlocked by the
    hardware); scalar instructions and s_nop count as wait states, every other instruction as one."""
    found = []
    for k, l in enumerate(ins):
        m = re.match(r"v_mfma_f32_32x32x16_bf16 v\[(\d+):(\d+)\]", l)
        if not m:
            continue
        lo, hi = int(m.group(1)), int(m.group(2))
        waited = 0
        for l2 in ins[k + 1:k + 1 + need]:
            if l2.startswith("v_mfma"):
                break
            if l2.startswith("s_nop"):
                waited += int(l2.split()[1]) + 1
                continue
            if not l2.startswith("s_"):
                regs = [int(x) for x in re.findall(r"\bv(\d+)\b", l2)]
                regs += [r for a, b in re.findall(r"v\[(\d+):(\d+)\]", l2) for r in range(int(a), int(b) + 1)]
                if any(lo <= r <= hi for r in regs) and waited < need:
                    found.append((l, l2, waited))
                    break
            waited += 1
            if waited >= need:
                break
    return found


def test_the_hazard_scan_sees_a_planted_early_copy():
    good = ["v_mfma_f32_32x32x16_bf16 v[8:23], v[0:3], v[4:7], v[8:23]", "s_nop 15", "s_nop 3", "v_mov_b32_e32 v40, v9"]
    assert early_reads_of_asm_mfma_results(good) == []
    chain = ["v_mfma_f32_32x32x16_bf16 v[8:23], v[0:3], v[4:7], v[8:23]",
             "v_mfma_f32_32x32x16_bf16 v[8:23], v[0:3], v[4:7], v[8:23]"]
    assert early_reads_of_asm_mfma_results(chain) == []
    bad = ["v_mfma_f32_32x32x16_bf16 v[8:23], v[0:3], v[4:7], v[8:23]", "s_nop 1", "v_mov_b64_e32 v[86:87], v[22:23]"]
    assert len(early_reads_of_asm_mfma_results(bad)) == 1
    builtin = ["v_mfma_f32_32x32x16_bf16 a[0:15], v[0:3], v[4:7], a[0:15]", "v_accvgpr_read_b32 v1, a0"]
    assert early_reads_of_asm_mfma_results(builtin) == []      # the compiler's own MFMAs: its business


def test_nothing_touches_an_asm_mfma_result_before_it_exists():
    text = backward_asm()
    names = [k for k in kernel_metadata(text) if "bwd_dkdv_kernel" in k or "bwd_dq_kernel" in k]
    assert len(names) == 6, names
    for name in names:
        ins = kernel_instructions(text, name)
        assert any(re.match(r"v_mfma_f32_32x32x16_bf16 v\[", l) for l in ins), name   # the asm form is in use
        assert early_reads_of_asm_mfma_results(ins) == [], name


def test_asm_mfma_kernels_have_no_vgpr_spills():
    text = backward_asm()
    meta = kernel_metadata(text)
    dkdv = {k: v for k, v in meta.items() if "bwd_dkdv_kernel" in k or "bwd_dq_kernel" in k}
    assert len(dkdv) == 6, meta
    for name, spills in dkdv.items():
        body = text[text.index("\n" + name + ":"):]
        body = body[:body.index(".end_amdhsa_kernel")]
        ins = [l.split()[0] for l in body.splitlines()
               if l.startswith("\t") and l.strip() and not l.strip().startswith((";", "."))]
        mfma = [i for i, op in enumerate(ins) if op.startswith("v_mfma")]
        scratch = [i for i, op in enumerate(ins) if op.startswith("scratch_")]
        assert mfma, name
        # nothing between the first MFMA and 64 instructions behind the last one (MFMA results are long
        # written by then), and no more than a handful of parked values altogether
        assert all(i < mfma[0] or i > mfma[-1] + 64 for i in scratch), (name, scratch, mfma[0], mfma[-1])
        assert spills <= 4, (name, spills)
        # nor copies between two sets of accumulator registers (the key-tile kernel issues every update
        # of dK / dV from one place so that the compiler keeps them in place)
        body = text[text.index("\n" + name + ":"):]
        body = body[:body.index(".end_amdhsa_kernel")]
        assert "v_accvgpr_mov" not in body, name


def test_the_forward_kernels_keep_their_registers():
    """What the forward takes in front of its loops comes out of its loops' registers: with a look-up of the tile
    order in it the head size 128 forms had gone from 246 and 250 registers to 252 and 256, and the one form with
    spills from 2 to 4; the 131072-token forward was 0.4 % longer."""
    text = device_asm("fwd.hip")
    regs = {m.group(1): int(m.group(2)) for m in
            re.finditer(r"\.name:\s+(\S+fwd_kernel\S+)\n(?:.*\n)*?\s+\.vgpr_count:\s+(\d+)", text)}
    spills = {k: v for k, v in kernel_metadata(text).items() if "fwd_kernel" in k}
    assert len(regs) == len(spills) == 9, (regs, spills)
    for name in regs:
        if "Li128ELi128E" in name:
            assert regs[name] <= 250, (name, regs[name])
        assert spills[name] <= (2 if "Li192ELi128ELi1ELi1E" in name else 0), (name, spills[name])


def test_the_forward_kernels_of_one_item_keep_their_registers():
    """The kernels that packs of few rounds run: no spills, registers for eight wavefronts a compute unit, and at head size 64
    for three workgroups of four wavefronts (512 registers a lane in a SIMD, given out by eight)."""
    text = device_asm("fwd.hip")
    regs = {m.group(1): int(m.group(2)) for m in
            re.finditer(r"\.name:\s+(\S+fwd_direct_kernel\S+)\n(?:.*\n)*?\s+\.vgpr_count:\s+(\d+)", text)}
    spills = {k: v for k, v in kernel_metadata(text).items() if "fwd_direct_kernel" in k}
    assert len(regs) == len(spills) == 9 and not any(spills.values()), (regs, spills)
    for name in regs:
        assert regs[name] <= (168 if "Li64ELi64ELi1ELi1E" in name else 256), (name, regs[name])


@pytest.mark.parametrize("source,kernels", [("fwd.hip", 18), ("bwd.hip", 13)])
def test_no_store_of_whole_rows_stands_in_a_loop_over_descriptors(source, kernels):
    """A buffer store takes its descriptor from scalar registers.  Where the compiler has part of it in vector registers it
    puts every such store into a loop over the values that the lanes might have, with a wait for the LDS read in each: all 4 to 12
    stores at the end of an item of the forward and of dQ had one."""
    text = device_asm(source)
    names = [n for n in kernel_metadata(text) if re.search(r"fwd_kernel|fwd_direct_kernel|bwd_dq|bwd_dkdv|bwd_both", n)]
    names = [n for n in names if "reduce" not in n]
    assert len(names) == kernels, names
    stores = 0
    for name in names:
        ins = kernel_instructions(text, name)
        for i, l in enumerate(ins):
            if l.startswith("buffer_store"):
                stores += 1
                assert not any(x.startswith("s_cbranch_execnz") for x in ins[i + 1:i + 5]), (name, ins[i:i + 5])
    assert stores >= kernels


@pytest.mark.parametrize("form", ["Li2ELi1E", "Li1ELi2E"])
def test_the_forwards_hot_loop_reloads_few_spilled_scalars(form):
    """Head size 128, eight wavefronts: the loop over pairs of unmasked tiles (64 MFMAs, some 1300 instructions) had 14
    and 16 such reloads with one function that takes an item with or without queues, and a pack of 5515 tokens with
    12/3 heads was 4 % longer than with 4 of them."""
    text = device_asm("fwd.hip")
    name = next(m for m in re.findall(r"\n(_ZN3hbp\d+fwd_kernel\w+):", text) if "ILi128ELi128E" + form in m)
    body = text[text.index("\n" + name + ":"):]
    lines = body[:body.index("s_endpgm")].splitlines()
    labels = {m.group(1): i for i, m in enumerate(re.match(r"(\.LBB\w+):", l) for l in lines) if m}
    loops = []
    for i, line in enumerate(lines):
        m = re.search(r"\ts_c?branch\w*\s+(\.LBB\w+)", line)
        if m and labels.get(m.group(1), i) < i:
            loop = [l for l in lines[labels[m.group(1)]:i + 1] if re.match(r"\t[a-z]", l)]
            if len(loop) < 1800 and sum("v_mfma" in l for l in loop) == 64:
                loops.append(sum("v_readlane" in l for l in loop))
    assert len(loops) == 1 and loops[0] <= 4, loops


def test_the_loss_kernels_keep_a_row_in_registers_without_spills():
    """A reload inside the loop over rows waits for the gradient stores of the row before (one counter, in order).
    With the planned range of rows in vector registers the longest rows (20 chunks, gradient) had one."""
    spills = {k: v for k, v in kernel_metadata(device_asm("loss.hip")).items() if "ce_main_kernel" in k}
    assert len(spills) == 76 and not any(spills.values()), {k: v for k, v in spills.items() if v}


def test_no_loss_workgroup_is_launched_beyond_those_that_fit():
    """The main kernel's grid is what the chip holds at once: a workgroup more than a compute unit's LDS has room for (given
    out in pieces of 1280 bytes of its 160 KB) would begin with its share of the rows when the others have ended.  The
    kernel's own arrays are taken from what the compiler gave them; where no rows are dealt, the rows' numbers are not among
    them (an LDS read a row instead of an addition: 1 % of 2500 rows of 4096)."""
    import launch_rules as rules
    kernels = [(tuple(int(x) for x in m.group(2, 3, 4, 5)), int(m.group(1))) for m in
               re.finditer(r"\.group_segment_fixed_size: (\d+)\n(?:(?!\s+\.name:).*\n)*\s+\.name:\s+\S+ce_main_kernelILi(\d+)ELi(\d+)ELb(\d)ELb(\d)E",
                           device_asm("loss.hip"))]
    assert len({k for k, _ in kernels}) == len(kernels) == 76
    for (threads, chunks, hold, grad), own in kernels:
        assert own <= rules.cross_entropy_own_lds(threads, chunks, hold, grad) <= own + 64, (threads, chunks, hold, grad, own)
        for n_samples in (1, 63, 1023):
            for T in list(range(512, 131073, 512)) + [131073]:
                plan = rules.cross_entropy_plan_lds(T, n_samples) if T <= 131072 else 0
                fit = 160 * 1024 // (-(-(plan + own) // 1280) * 1280)
                launched = rules.cross_entropy_launched_per_cu(threads, chunks, hold, grad, T, n_samples)
                assert launched <= fit, (threads, chunks, hold, grad, T, n_samples, launched, fit)


@pytest.mark.parametrize("source,least", [("fwd.hip", 16), ("bwd.hip", 11)])
def test_the_race_hunting_build_waits_for_all_copies_of_an_items_rows(source, least):
    """The release build waits for an item's rows by a count of copies.  Were a count too high, the build that it is compared
    with would have to differ: it waits for all of them in front of the first LDS read behind every such count."""
    def counted_waits(text):
        out = []
        for name in kernel_metadata(text):
            ins = kernel_instructions(text, name)
            for i, l in enumerate(ins):
                m = re.match(r"s_waitcnt vmcnt\((\d+)\)$", l)
                copies = [k for k in range(max(0, i - 400), i) if re.match(r"buffer_load_dwordx4 .*lds", ins[k])]
                read = next((k for k in range(i, min(i + 120, len(ins))) if ins[k].startswith("ds_read_b128")), None)
                in_a_step = any(x.startswith("v_mfma") for x in ins[max(0, i - 300):i])
                if m and int(m.group(1)) and copies and read is not None and not in_a_step:
                    out.append((name, i, any("vmcnt(0)" in x for x in ins[copies[-1]:read])))
        return out
    release, hunting = counted_waits(device_asm(source)), counted_waits(device_asm(source, ["-DHBP_RACE_HUNT"]))
    assert sum(not full for _, _, full in release) >= least, release
    assert len(hunting) >= least and all(full for _, _, full in hunting), hunting
