"""A property of the generated code that the source relies on and cannot express (CPU only: hipcc cross-compiles).

attn_fwd64 reads every V fragment with two transposed LDS reads whose results land asynchronously; the source
joins the two halves into the register quadruple of an MFMA operand right at the reads.  That is only correct if
the compiler makes the reads write the quadruple's halves directly: a register copy between a read and the
wait for it would copy stale data.  The check: in the compiled kernel every pair of consecutive transposed reads
fills two adjacent register pairs, and that quadruple is read by an MFMA as it stands."""
import os
import re
import shutil
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not found")
def test_v_fragments_are_read_into_the_mfma_operand_registers():
    from paper_2409_09086_amd.build import CSRC, FLAGS
    with tempfile.TemporaryDirectory() as tmp:
        asm = os.path.join(tmp, "attn_mfma64.s")
        subprocess.run(["hipcc", *[f for f in FLAGS if f != "-fPIC"], "-I" + os.path.join(ROOT, "include"), "-S",
                        "--cuda-device-only", os.path.join(CSRC, "attn_mfma64.hip"), "-o", asm],
                       check=True, capture_output=True)
        lines = open(asm).read().splitlines()
    reads = [int(m.group(1)) for l in lines for m in [re.search(r"ds_read_b64_tr_b16 v\[(\d+):(\d+)\]", l)] if m]
    assert len(reads) >= 64 and len(reads) % 2 == 0, len(reads)
    quads = set()
    for lo, hi in zip(reads[0::2], reads[1::2]):
        assert hi == lo + 2, "the two halves of a V fragment do not fill one register quadruple: v%d, v%d" % (lo, hi)
        quads.add((lo, lo + 3))
    operands = set()
    for l in lines:
        m = re.search(r"v_mfma_f32_32x32x16_bf16 a\[\d+:\d+\], v\[(\d+):(\d+)\], v\[", l)
        if m:
            operands.add((int(m.group(1)), int(m.group(2))))
    assert operands, "no O += V^T P^T product found"
    missing = sorted(quads - operands)
    assert not missing, "V fragments that no MFMA reads from the registers they were read into: %s" % missing


def device_code(src):
    from paper_2409_09086_amd.build import CSRC, FLAGS
    with tempfile.TemporaryDirectory() as tmp:
        asm = os.path.join(tmp, "k.s")
        subprocess.run(["hipcc", *[f for f in FLAGS if f != "-fPIC"], "-S", "--cuda-device-only", os.path.join(CSRC, src), "-o", asm],
                       check=True, capture_output=True)
        text = open(asm).read()
    kernels = {}
    for m in re.finditer(r"^(_Z\w+):(.*?)^\s*\.section", text, re.M | re.S):
        kernels[m.group(1)] = m.group(2)
    scratch = {m.group(1): int(m.group(2)) for m in re.finditer(r"\.set (_Z\w+)\.private_seg_size, (\d+)", text)}
    return kernels, scratch


def registers(operands, kinds="v"):
    """Vector registers (accumulation registers with kinds "a") named in an operand list."""
    out = set()
    for m in re.finditer(r"\b([%s])(?:\[(\d+):(\d+)\]|(\d+)\b)" % kinds, operands):
        lo = int(m.group(2) or m.group(4))
        out.update((m.group(1), r) for r in range(lo, int(m.group(3) or lo) + 1))
    return out


def reads_touched_too_early(body, kinds="v"):
    """Vector LDS reads of asm statements that do not wait themselves: (how many there are, those whose registers an
    instruction names, or that a branch or label follows, before a wait that covers them).  kinds "a": reads into accumulation
    registers only."""
    pending, found, bad, in_asm = [], 0, [], False      # pending: LDS and scalar operations in issue order, a read's registers or None
    lines = body.splitlines()
    for i, line in enumerate(lines):
        if "#ASMSTART" in line or "#ASMEND" in line:
            in_asm = "#ASMSTART" in line
            continue
        code = line.split(";")[0].strip()
        if not code or code.startswith("."):
            if re.match(r"\.L\w+:", code) and any(p for p in pending):
                bad.append((i, code))
            continue
        op, _, args = code.partition(" ")
        if op == "s_waitcnt":
            m = re.search(r"lgkmcnt\((\d+)\)", args)
            if m:
                pending = pending[len(pending) - min(len(pending), int(m.group(1))):]
            continue
        if op.startswith("s_cbranch") or op == "s_branch":
            if any(p for p in pending):
                bad.append((i, code))
            continue
        names = registers(args, kinds)
        if any(p and p & names for p in pending):
            bad.append((i, code))
        target = registers(args.split(",")[0], kinds) if op.startswith("ds_read") and in_asm else None
        if target:
            found += 1
            pending.append(target)
        elif op.startswith(("ds_", "s_load", "s_buffer_load", "s_memrealtime")):
            pending.append(None)
    return found, bad


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not found")
@pytest.mark.parametrize("src,name,instances", [("attn_rows.hip", "attn_rows_kernel", 12), ("attn_rows64.hip", "attn_rows64_kernel", 2),
                                                ("attn_f32.hip", "attn_f32_kernel", 4)])
def test_lds_reads_are_not_touched_before_the_wait_that_covers_them(src, name, instances):
    """The kernels that wait for their LDS reads by hand: the compiler takes a read's registers as written at once, and must
    have no copy, spill or use of them before the wait.  (LDS reads return in order; a wait for n leaves the n newest operations.)"""
    kernels, scratch = device_code(src)
    mine = {k: v for k, v in kernels.items() if name in k}
    assert len(mine) == instances, sorted(kernels)
    for k, body in mine.items():
        found, bad = reads_touched_too_early(body)
        assert found >= 8 and not bad, (k, found, bad[:5])
    if name == "attn_rows64_kernel":
        # no register to spare: a spill's reload in the loop would wait for every load in flight
        assert all(scratch[k] == 0 for k in mine), scratch


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not found")
def test_attn_fwd64_reads_its_queries_into_the_registers_of_its_products():
    """attn_fwd64's query fragments go from LDS into accumulation registers, waited for by hand (its other reads are checked above and by
    the results: they stay in flight over the side path).  All of them, sixteen in each instance, none touched before the wait; and no
    instance, the one for cut key ranges fills all 512 registers, keeps anything in scratch."""
    kernels, scratch = device_code("attn_mfma64.hip")
    mine = {k: v for k, v in kernels.items() if "attn_fwd64_kernel" in k}
    assert len(mine) == 2, sorted(kernels)
    for k, body in mine.items():
        found, bad = reads_touched_too_early(body, "a")
        assert found == 16 and not bad, (k, found, bad[:5])
        assert scratch[k] == 0, scratch


def test_the_check_finds_a_read_that_is_touched_too_early():
    read = "\t;;#ASMSTART\n\tds_read_b128 v[4:7], v1 offset:0\n\t;;#ASMEND\n"
    assert reads_touched_too_early(read + read.replace("4:7", "8:11") + "\ts_waitcnt lgkmcnt(1)\n\tv_add_f32_e32 v0, v4, v7\n") == (2, [])
    for early in ("\tv_mov_b32_e32 v0, v5\n", "\tscratch_store_dwordx4 off, v[4:7], off offset:16\n", "\ts_cbranch_scc1 .LBB0_1\n",
                  "\ts_waitcnt lgkmcnt(1)\n\tv_mov_b32_e32 v0, v5\n"):
        assert len(reads_touched_too_early(read + early)[1]) == 1
    acc = read.replace("v[4:7]", "a[4:7]")
    assert reads_touched_too_early(acc + "\ts_waitcnt lgkmcnt(0)\n\tv_accvgpr_read_b32 v0, a5\n", "a") == (1, [])
    for early in ("\tv_accvgpr_read_b32 v0, a5\n", "\tv_mfma_f32_32x32x16_bf16 v[0:15], v[16:19], a[4:7], 0\n", "\ts_branch .LBB0_1\n"):
        assert len(reads_touched_too_early(acc + early, "a")[1]) == 1
