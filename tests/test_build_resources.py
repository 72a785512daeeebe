"""The attention kernels run at 2 waves per SIMD with all 256 registers in use: a register spill in
a hot loop costs a scratch round trip per tile (and, because vector-memory loads return in order, a
wait for the tile prefetch in flight).  This test compiles the kernels with the compiler's resource
remarks and fails if a production kernel spills or loses its occupancy.  CPU only: hipcc cross-compiles."""
import functools
import os
import re
import shutil
import subprocess
import tempfile

import pytest

from paper_2603_00040_amd import build as B

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not on PATH")


@functools.lru_cache(maxsize=None)
def _resources(src):
    with tempfile.TemporaryDirectory() as tmp:
        r = subprocess.run(["hipcc", *B.FLAGS, "-Rpass-analysis=kernel-resource-usage", "-c",
                            os.path.join(B.CSRC, src), "-o", os.path.join(tmp, "x.o")],
                           capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    out, cur = {}, None
    for line in r.stderr.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            cur = out.setdefault(m.group(1), {})
            continue
        m = re.search(r"remark:\s+(VGPRs Spill|SGPRs Spill|Occupancy \[waves/SIMD\]|ScratchSize \[bytes/lane\]): (\d+)", line)
        if m and cur is not None:
            cur[m.group(1)] = int(m.group(2))
    return out


def _check(kernels, pattern, expect_count, spill_free=True):
    hit = {k: v for k, v in kernels.items() if re.search(pattern, k)}
    assert len(hit) == expect_count, (pattern, sorted(kernels))
    for name, res in hit.items():
        if spill_free:
            assert res["VGPRs Spill"] == 0 and res["SGPRs Spill"] == 0 and res["ScratchSize [bytes/lane]"] == 0, (name, res)
        assert res["Occupancy [waves/SIMD]"] >= 2, (name, res)
    return hit


def _scratch_in_inner_loops(src, pattern):
    """For every kernel of `src` whose mangled name matches: the scratch instructions that lie inside an innermost loop
    (from the block annotations of the compiler's assembly listing).  A spill outside the loops costs a few instructions
    once; one inside a key loop costs a scratch round trip per tile."""
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "x.s")
        r = subprocess.run(["hipcc", *B.FLAGS, "-S", "--cuda-device-only", os.path.join(B.CSRC, src), "-o", out],
                           capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
        text = open(out).read().splitlines()
    found, cur, inner, in_inner = {}, None, set(), False
    for line in text:
        m = re.match(r"^(_Z\w+):", line)
        if m:
            cur = m.group(1) if re.search(pattern, m.group(1)) else None
            if cur:
                found[cur] = []
            inner, in_inner = set(), False
            continue
        if cur is None:
            continue
        m = re.match(r"^(\.LBB\d+_\d+):(.*)", line)
        if m:
            label, note = m.group(1), m.group(2)
            if "Inner Loop Header" in note:
                inner.add(label.lstrip("."))
                in_inner = True
            else:
                h = re.search(r"in Loop: Header=(BB\d+_\d+)", note)
                in_inner = bool(h) and ("L" + h.group(1)) in {"L" + x.lstrip("L") for x in inner}
            continue
        if re.match(r"^; %bb\.\d+:", line):
            h = re.search(r"in Loop: Header=(BB\d+_\d+)", line)
            in_inner = bool(h) and ("L" + h.group(1)) in {"L" + x.lstrip("L") for x in inner}
            continue
        if in_inner and "scratch_" in line:
            found[cur].append(line.strip())
    return found


def test_forward_kernels_do_not_spill():
    k = _resources("fwd.hip")
    # fwd_kernel<D, TRAIN, CAUSAL, DUMP, PQ, VARLEN>: every production variant (DUMP = false), d = 64 and 128, the three block
    # forms of phi(P); the bf16 P-tilde of the mixed recipe (inference only); the per-sequence lengths of the paged forward
    _check(k, r"fwd_kernelILi(64|128)ELb[01]ELb0ELb0ELi[012]ELb0E", 12)
    _check(k, r"fwd_kernelILi(64|128)ELb0ELb0ELb0ELi3ELb0E", 2)
    _check(k, r"fwd_kernelILi(64|128)ELb0ELb0ELb0ELi0ELb1E", 2)
    # Causal variants: a workgroup takes two query tiles one after the other, and the compiler parks a few values that only
    # the set-up and the wind-down of a tile use (the lane number, two constants) in scratch across the key loop.  What must
    # not happen is a scratch access inside the key loop.
    causal = r"fwd_kernelILi(64|128)ELb[01]ELb1ELb0ELi[0123]ELb[01]E"      # 12 + 2 (bf16 P-tilde) + 2 (per-sequence lengths)
    hit = _check(k, causal, 16, spill_free=False)
    # (scalar registers parked in lanes of a vector register cost no memory access: up to 16 of them, mostly the MX variants,
    #  which carry the addresses of two more operand arrays)
    assert all(v["VGPRs Spill"] <= 8 and v["SGPRs Spill"] <= 16 for v in hit.values()), hit
    inner = _scratch_in_inner_loops("fwd.hip", causal)
    assert len(inner) == 16 and all(not v for v in inner.values()), {n: v for n, v in inner.items() if v}


def test_backward_kernels_do_not_spill():
    k = _resources("bwd.hip")
    _check(k, r"bwd_dq_kernelILi(64|128)ELb[01]ELb[01]ELi[48]E", 16)    # <D, CAUSAL, scores on the FP4 instruction (MX), waves>
    # bwd_dkdv_kernel<D, CAUSAL, COUNT, PQ>: the measurement (COUNT) and ablation (PQ = 0) variants are exempt
    _check(k, r"bwd_dkdv_kernelILi(64|128)ELb[01]ELb0ELi[123]ELi[48]E", 24)   # 12 of 4 waves, 12 of 8


def test_decode_kernels_do_not_spill():
    k = _resources("decode.hip")
    hit = _check(k, r"decode_kernelILi(64|128)ELb[01]E", 4, spill_free=False)
    # no scratch memory; scalar registers parked in vector lanes are tolerated (the kernel takes twenty arguments)
    assert all(v["VGPRs Spill"] == 0 and v["ScratchSize [bytes/lane]"] == 0 for v in hit.values()), hit


def test_mx_forward_kernels_do_not_spill():
    k = _resources("mx.hip")
    # fwd_mx_kernel<D, CAUSAL, FP8PV, KVM>: 8 contiguous variants, the 4 paged and the 4 block-sparse ones (FP4 only)
    _check(k, r"fwd_mx_kernelILi(64|128)ELb[01]ELb[01]ELi[012]E", 16)
    # fwd_mx_decode_kernel<D, CAUSAL, NP = 1>: two workgroups per CU
    _check(k, r"fwd_mx_decode_kernelILi(64|128)ELb[01]ELi1E", 4)


def test_four_wave_forward_kernels_do_not_spill():
    # fwd_narrow_kernel<D, TRAIN, CAUSAL, PQ, VARLEN>: the forward of every problem that does not fill the chip with eight-wave workgroups
    k = _resources("fwd.hip")
    _check(k, r"fwd_narrow_kernelILi(64|128)ELb[01]ELb[01]ELi[012]ELb0E", 24)
    _check(k, r"fwd_narrow_kernelILi(64|128)ELb0ELb[01]ELi3ELb0E", 4)
    _check(k, r"fwd_narrow_kernelILi(64|128)ELb0ELb[01]ELi0ELb1E", 4)
    assert len([n for n in k if "fwd_narrow_kernel" in n]) == 32


def test_joint_backward_kernels_do_not_spill():
    # bwd_joint_kernel<D, CAUSAL, PQ, COUNT>: the backward of all but the largest problems; the measurement variants (COUNT) are exempt
    k = _resources("bwd.hip")
    _check(k, r"bwd_joint_kernelILi(64|128)ELb[01]ELi[123]ELb0E", 12)
    _check(k, r"dkdv_reduce_kernelILi(64|128)ELb[01]E", 4)


def test_few_rows_backward_kernels_do_not_spill():
    # bwd_few_kernel<D, CAUSAL>: operands of four tiles at a time; one workgroup, of a wavefront per SIMD, on a compute unit
    hit = {n: v for n, v in _resources("bwd.hip").items() if re.search(r"bwd_few_kernelILi(64|128)ELb[01]E", n)}
    assert len(hit) == 4
    assert all(v["VGPRs Spill"] == 0 and v["SGPRs Spill"] == 0 and v["ScratchSize [bytes/lane]"] == 0 for v in hit.values()), hit


def test_backward_of_d64_leaves_room_for_three_wavefronts():
    # (a SIMD has 512 registers; with more than 168 each, two)
    hit = _check(_resources("bwd.hip"), r"bwd_joint_kernelILi64ELb[01]ELi[123]ELb0E", 6)
    assert all(v["Occupancy [waves/SIMD]"] >= 3 for v in hit.values()), hit


def test_preparing_kernels_keep_off_scratch_memory():
    # scalar registers parked in lanes of a vector register cost no memory access: the backward's group carries the addresses of
    # nine arrays beside its loop bounds
    for src, pattern, n in (("prep.hip", r"(prep_group_kernelI|quantize_kernelE|kv_page_write_kernelI)", 9),
                            ("mxprep.hip", r"(mx_group_kernelI|mx_q_kernelI)", 10), ("decode.hip", r"decode_(prepare|merge)_kernelI", 4)):
        hit = _check(_resources(src), pattern, n, spill_free=False)
        assert all(v["VGPRs Spill"] == 0 and v["ScratchSize [bytes/lane]"] == 0 and v["SGPRs Spill"] <= 48 for v in hit.values()), hit
        assert all(v["Occupancy [waves/SIMD]"] >= 5 for v in hit.values()), hit


@pytest.mark.parametrize("src", ["fwd.hip", "mx.hip"])
def test_no_lds_read_is_in_flight_at_a_barrier_of_the_forward(src):
    """The forward's barriers are bare ones (no fence): behind a barrier another wave copies the next tile over the one that was just
    read, or, where waves share key tiles, writes its P and row maxima over them, so every LDS read has to have arrived before it (listing
    read from top to bottom, reads minus what the waits leave).  In the four-wave kernels the second barrier is the one behind the scores of
    tile 0: all of their products stand in front of it."""
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "x.s")
        r = subprocess.run(["hipcc", *B.FLAGS, "-S", "--cuda-device-only", os.path.join(B.CSRC, src), "-o", out], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
        text = open(out).read().splitlines()
    seen, cur = {}, None
    for line in (l.strip() for l in text):
        m = (re.match(r"^_ZN2aq\d+(fwd_(?:narrow_|split_)?kernel)ILi(64|128)E\S*?(?:ELi|ELb[01]ELi)([0-3])ELb[01]E\S*:", line)
             or re.match(r"^_ZN2aq\d+(fwd_mx_split_kernel)ILi(64|128)E\S*?ELi([0-2])E\S*:", line))
        if m:
            cur, reads, products = line, 0, 0
            seen[cur] = (m.group(1), int(m.group(2)), int(m.group(3)), [])
        elif line.startswith(".Lfunc_end"):
            cur = None
        elif cur and line.startswith("ds_read"):
            reads += 1
        elif cur and line.startswith("v_mfma"):
            products += 1
        elif cur and line.startswith("s_waitcnt") and "lgkmcnt" in line:
            reads = min(reads, int(re.search(r"lgkmcnt\((\d+)\)", line).group(1)))
        elif cur and line.startswith("s_barrier"):
            seen[cur][3].append((reads, products))
            products = 0
    if src == "mx.hip":
        assert len(seen) == 16
    else:
        assert len([k for k in seen if "narrow" in k]) == 32 and len([k for k in seen if "split" in k]) == 24 and len(seen) > 88
    for name, (kind, d, pq, barriers) in seen.items():
        assert barriers and all(b[0] == 0 for b in barriers), (name, barriers)
        if kind == "fwd_narrow_kernel":
            assert barriers[1][1] == (2 * d // 64 if pq == 1 else 2 * d // 16), (name, barriers)      # (MX: the FP4 instruction)


def test_split_forward_kernels_do_not_spill():
    # fwd_split_kernel<D, TRAIN, CAUSAL, PQ, VARLEN>: the forward of few query rows (no two-level variant)
    k = _resources("fwd.hip")
    _check(k, r"fwd_split_kernelILi(64|128)ELb[01]ELb[01]ELi[01]ELb0E", 16)
    _check(k, r"fwd_split_kernelILi(64|128)ELb0ELb[01]ELi(3ELb0|0ELb1)E", 8)
    assert len([n for n in k if "fwd_split_kernel" in n]) == 24


def test_decode_kernels_without_a_queue_keep_off_scratch_memory():
    _check(_resources("decode.hip"), r"decode_(scores_kernelILi(64|128)ELb[01]|values_kernelILi(64|128))E", 6)


def test_mx_decode_kernels_in_chunks_do_not_spill():
    _check(_resources("mx.hip"), r"mx_decode_(p|max)_kernelILi(64|128)ELb[01]E", 8)
    _check(_resources("mx.hip"), r"mx_decode_pv_kernelILi(64|128)E", 2)


def test_split_mx_forward_kernels_do_not_spill():
    # fwd_mx_split_kernel<D, CAUSAL, FP8PV, KVM>: contiguous in both recipes, paged and block-sparse
    _check(_resources("mx.hip"), r"fwd_mx_split_kernelILi(64|128)ELb[01]E(Lb0ELi[012]|Lb1ELi0)E", 16)


def _registers(operand):
    m = re.match(r"[-|]*v(?:\[(\d+):(\d+)\]|(\d+))\|?$", operand)
    return range(0) if not m else range(int(m.group(1)), int(m.group(2)) + 1) if m.group(1) else range(int(m.group(3)), int(m.group(3)) + 1)


def _reads_without_settling(src, pattern, suspect):
    """For every kernel whose mangled name matches: its vector instructions that read the result of a product although no wait written in
    the source (s_nop in inline assembly) stands in between, out of those that suspect(product, in another block, in inline assembly)
    picks, unless another of their operands has been made from the same product by instructions that the compiler counts for.  The
    listing is read from top to bottom; after 20 instructions every product has arrived."""
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "x.s")
        r = subprocess.run(["hipcc", *B.FLAGS, "-S", "--cuda-device-only", os.path.join(B.CSRC, src), "-o", out], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
        text = open(out).read().splitlines()
    found, cur, written, made, at, block, in_asm, settled = {}, None, {}, {}, 0, 0, False, 0
    for line in (l.strip() for l in text):
        m = re.match(r"^(_Z\w+):", line)
        if m:
            cur = m.group(1) if re.search(pattern, m.group(1)) else None
            written, made, at, block, settled = {}, {}, 0, 0, 0
            if cur:
                found[cur] = []
        elif line.startswith((".LBB", "; %bb")):
            block += 1
        elif "ASMSTART" in line or "ASMEND" in line:
            in_asm = "ASMSTART" in line
        elif cur and line and line[0] not in ";.":
            op, _, rest = line.partition(" ")
            operands = [t.strip().split(" ")[0] for t in rest.split(",")]
            at += int(operands[0]) + 1 if op == "s_nop" else 1
            if op == "s_nop" and in_asm:
                settled = at
            elif op.startswith("v_mfma"):
                written.update({reg: (at, block, op) for reg in _registers(operands[0])})
            elif op.startswith("v_"):
                sources = [reg for t in operands[1:] for reg in _registers(t)]
                beside = set().union(*(made.get(reg, set()) for reg in sources if reg not in written)) if sources else set()
                for reg in (reg for reg in sources if reg in written):
                    when, where, product = written[reg]
                    if settled < when and at - when < 20 and when not in beside and suspect(product, block != where, in_asm):
                        found[cur].append((at - when, line))
                result = beside | {written[reg][0] for reg in sources if reg in written}
                for reg in _registers(operands[0]):
                    written.pop(reg, None)
                    made[reg] = result
    return found


def test_inline_assembly_of_the_split_forward_reads_settled_products():
    """The compiler counts the wait states between a product and its readers, but does not look into inline assembly (max_raw): in the kernel
    that has no barrier between the scores and the softmax, such a read has to wait in the source or depend on a counted one."""
    found = _reads_without_settling("fwd.hip", r"fwd_split_kernel", lambda product, other_block, in_asm: in_asm)
    assert len(found) == 24 and not any(found.values()), {k: v[:3] for k, v in found.items() if v}


@pytest.mark.parametrize("pattern,n", [(r"fwd_mx_split_kernelILi(64|128)ELb[01]ELb0E", 12), (r"fwd_mx_split_kernelILi(64|128)ELb[01]ELb1E", 4), (r"mx_decode_pv_kernel", 2)])
def test_products_that_another_block_reads_have_settled(pattern, n):
    """The rescaling of O reads the product of the tile in front in a block of its own: the wait states (FP4 operands 11, FP8 19) that
    the compiler puts there are in the listing.  Inline assembly reads no product that has not settled in the source."""
    found = _reads_without_settling("mx.hip", pattern, lambda product, other_block, in_asm: "scale" in product and (other_block or in_asm))
    need = 19 if "ELb1E" in pattern[-6:] else 11
    assert len(found) == n and all(when > need for reads in found.values() for when, _ in reads), {k: v[:3] for k, v in found.items() if v}
    assert not any("v_max_f32" in line for reads in found.values() for _, line in reads)
