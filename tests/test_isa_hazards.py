"""Static check of the compiled GEMM kernels (no GPU needed).

The tall tiles (256 and 288 rows) issue every MFMA through inline asm that names the register file of the
accumulator (AGPRs, and VGPRs for two token blocks of the 288-row tile), which the compiler's hazard
recogniser cannot see into.  Two things it would otherwise guarantee are checked here on the compiled code,
instruction by instruction and following branches: nothing but the next accumulating MFMA touches an MFMA's
result until it has been written (7 wait states after a 4-pass MFMA), and nothing writes an operand of an
asm MFMA in the wait states right before it.  Loads through inline asm are followed to the wait that covers them; stores
through inline asm are not allowed at all.
"""
import re

import pytest

NEED = 8           # wait states before anything else may touch the result (7 by the ISA tables, one to spare)
MFMA_PASSES = 4    # v_mfma_f32_16x16x32_bf16; the pipe takes the next MFMA when the previous one has gone through


def _regs(tok):
    """Registers named by an operand token, as (file, index) pairs: v7, v[2:5], a3, a[0:3]."""
    m = re.fullmatch(r"([va])\[(\d+):(\d+)\]", tok)
    if m:
        return {(m.group(1), r) for r in range(int(m.group(2)), int(m.group(3)) + 1)}
    m = re.fullmatch(r"([va])(\d+)", tok)
    return {(m.group(1), int(m.group(2)))} if m else set()


def _split(line):
    body = line.split(";")[0].strip()
    parts = body.split(None, 1)
    if not parts:
        return "", []
    return parts[0], ([t.strip() for t in re.split(r",\s*", parts[1])] if len(parts) > 1 else [])


def find_hazards(lines, agpr_too=False):
    """Returns (number of MFMAs checked, list of hazard descriptions).  Checked are the MFMAs with a VGPR
    destination and, with agpr_too, those with an AGPR destination as well (kernels that issue every MFMA
    through inline asm)."""
    labels = {}
    for i, l in enumerate(lines):
        m = re.match(r"(\.LBB\d+_\d+):", l)
        if m:
            labels[m.group(1)] = i
    pinned, bad = 0, []
    for i, l in enumerate(lines):
        op, ops = _split(l)
        if not op.startswith("v_mfma") or not ops:
            continue
        if not (ops[0].startswith("v") or (agpr_too and ops[0].startswith("a"))):
            continue
        pinned += 1
        dst = _regs(ops[0])
        work, seen = [(i + 1, 0, MFMA_PASSES)], set()
        while work:
            j, t, free = work.pop()
            while j < len(lines) and t < NEED:
                s = lines[j].strip()
                j += 1
                if not s or s.startswith(";") or s.startswith("."):
                    continue
                o, oo = _split(s)
                if o == "s_nop":
                    t += int(oo[0]) + 1
                    continue
                if o.startswith("v_mfma"):
                    t = max(t, free)
                    free = t + MFMA_PASSES
                    touched = set().union(*[_regs(x) for x in oo]) & dst
                    if touched and not (oo[0] == oo[3] and _regs(oo[0]) == dst):
                        bad.append(f"line {j}: MFMA touches the result of line {i + 1} after {t} states: {s}")
                    t += 1
                    continue
                touched = set()
                for x in oo:
                    for tok in re.findall(r"[va]\[\d+:\d+\]|\b[va]\d+\b", x):
                        touched |= _regs(tok)
                if touched & dst:
                    bad.append(f"line {j}: touches the result of line {i + 1} after {t} states: {s}")
                    break
                if o == "s_endpgm":
                    break
                if o == "s_branch":
                    if oo[0] in seen:
                        break
                    seen.add(oo[0])
                    j = labels[oo[0]]
                elif o.startswith("s_cbranch") and oo[0] not in seen:
                    seen.add(oo[0])
                    work.append((labels[oo[0]], t + 1, free))
                t += 1
    return pinned, bad


WRITE_TO_MFMA = 4  # wait states between an instruction that writes a register and an asm MFMA that reads it


def find_late_writers(lines):
    """The other direction, for the MFMAs issued through inline asm (between the compiler's ASMSTART / ASMEND
    marks): an instruction other than an MFMA that writes one of their operand registers must lie at least
    WRITE_TO_MFMA wait states before them (the compiler inserts those states for the MFMAs it knows).  Scans
    back inside the basic block; loads are waited for explicitly and are not instructions of this kind."""
    bad, checked, in_asm = [], 0, False
    for i, l in enumerate(lines):
        s = l.strip()
        if s.startswith(";;#ASMSTART"):
            in_asm = True
            continue
        if s.startswith(";;#ASMEND"):
            in_asm = False
            continue
        op, ops = _split(s)
        if not in_asm or not op.startswith("v_mfma"):
            continue
        checked += 1
        reads = set().union(*[_regs(x) for x in ops[1:]])
        t, j = 0, i - 1
        while j >= 0 and t < WRITE_TO_MFMA:
            p = lines[j].strip()
            j -= 1
            if not p or p.startswith(";") or p.startswith("."):
                if re.match(r"\.LBB\d+_\d+:", p):
                    break
                continue
            o, oo = _split(p)
            if o == "s_nop":
                t += int(oo[0]) + 1
                continue
            if o.startswith("v_") and not o.startswith("v_mfma") and oo and (_regs(oo[0]) & reads):
                bad.append(f"line {j + 2}: writes an operand of the asm MFMA at line {i + 1} only {t} states before it: {p}")
                break
            t += 1
    return checked, bad


_COPIES = ("v_mov_b", "v_accvgpr_", "v_swap", "scratch_store", "buffer_store", "global_store", "flat_store", "ds_write")


def find_touched_before_arrival(lines):
    """The weight loads are inline asm too (global_load_dwordx4 between ASMSTART / ASMEND), waited for with
    explicit counts: the compiler does not know that their destination registers are not valid yet and could
    copy or reuse them.  From every such load, walk forward along both sides of every branch to an s_waitcnt whose
    vmcnt is no larger than the number of vector-memory instructions issued since, and flag what names a
    destination register before that.  The loads of a K step are in flight across its barrier and landed before the
    next one, so a path ends at its second barrier; and at the asm that computes the lane anew, which opens the
    epilogue and the code of another tile height.  Past the first barrier only what copies a destination
    register is flagged -- moves, also between the register files, and stores, which is what a register allocator puts
    there: the conditions of the last K steps are not followed, and on paths that cannot be taken the registers are free
    for other uses.
    Returns (loads checked, loads followed past a barrier, hazards)."""
    labels, ins, in_asm = {}, [], False
    for i, l in enumerate(lines):
        m = re.match(r"(\.LBB\d+_\d+):", l)
        if m:
            labels[m.group(1)] = i
        p = l.strip()
        if p.startswith(";;#ASM"):
            in_asm = p.startswith(";;#ASMSTART")
        op, ops = _split(p)
        if not op or op.endswith(":") or p.startswith((";", ".")):
            ins.append(None)
            continue
        regs = set()
        for x in ops:
            for tok in re.findall(r"[va]\[\d+:\d+\]|\b[va]\d+\b", x):
                regs |= _regs(tok)
        copied = regs if "store" in op or op.startswith(("ds_write", "v_swap")) else regs - _regs(ops[0] if ops else "")
        ins.append((op, copied if op.startswith(_COPIES) else set(), regs, in_asm, p))
    checked, crossed, bad = 0, 0, []
    for i, load in enumerate(ins):
        if load is None or not load[3] or not load[0].startswith("global_load_dwordx4"):
            continue
        checked += 1
        dst = _regs(_split(load[4])[1][0])
        paths, seen, past, found = [(i + 1, 0, 0)], set(), False, None
        while paths and found is None:
            j, later, barriers = paths.pop()
            while j < len(ins):
                at, j = ins[j], j + 1
                if at is None:
                    continue
                op, copied, regs, asm, p = at
                if op == "s_waitcnt":
                    m = re.search(r"vmcnt\((\d+)\)", p)
                    if m and int(m.group(1)) <= later:
                        break
                    continue
                if op == "s_barrier":
                    barriers, past = barriers + 1, True
                    if barriers == 2:
                        break
                    continue
                if op == "s_endpgm" or (asm and op.startswith("v_mbcnt")):
                    break
                if (regs if barriers == 0 else copied) & dst:
                    found = f"line {j}: names a register of the load at line {i + 1} before it has been waited for: {p}"
                    break
                if op.startswith(("global_", "buffer_", "scratch_", "flat_")):
                    later = min(later + 1, 63)  # the counter's largest value
                if op == "s_branch":
                    j = labels[p.split()[1]]
                    if (j, later, barriers) in seen:
                        break
                    seen.add((j, later, barriers))
                elif op.startswith("s_cbranch"):
                    for state in ((labels[p.split()[1]], later, barriers), (j, later, barriers)):
                        if state not in seen:
                            seen.add(state)
                            paths.append(state)
                    break
        crossed += past
        if found is not None:
            bad.append(found)
    return checked, crossed, bad


def find_asm_stores(lines):
    """Stores to memory issued through inline asm.  A vector instruction that overwrites the data registers of a store of
    more than 64 bits needs two wait states behind it; the compiler inserts them for the stores it knows, not for these."""
    bad, in_asm = [], False
    for i, l in enumerate(lines):
        s = l.strip()
        if s.startswith(";;#ASM"):
            in_asm = s.startswith(";;#ASMSTART")
        elif in_asm and re.match(r"(global|flat|buffer|scratch)_store", s):
            bad.append(f"line {i + 1}: store the compiler cannot see into: {s}")
    return bad


def test_lint_flags_an_asm_store():
    st = "\tglobal_store_dwordx4 v64, v[40:43], s[22:23] sc1"
    assert len(find_asm_stores(["\t;;#ASMSTART", st, "\t;;#ASMEND", "\tv_add_u32_e32 v40, 8, v1"])) == 1
    assert find_asm_stores([st, "\t;;#ASMSTART", "\ts_nop 0", "\t;;#ASMEND", st]) == []


@pytest.mark.parametrize("unit,heights", [("moe_gemm_plain_stream", {288}), ("moe_gemm_swiglu_stream", {288}),
                                            ("moe_gemm_plain", set()), ("moe_gemm_swiglu", set())])
def test_stores_of_device_scope_stand_in_the_tall_streaming_kernels_only(unit, heights, gemm_unit_asm):
    kernel, scoped = None, set()
    for line in gemm_unit_asm[unit]:
        m = re.match(r"(_Z\w*grouped_gemm_kernelILi(\d+)E\w*):", line)
        if m:
            kernel = int(m.group(2))
        op, ops = _split(line)
        if op.startswith("global_store") and " sc1" in line:
            assert op == "global_store_dwordx4"
            scoped.add(kernel)
    assert scoped == heights


def test_lint_flags_a_register_used_before_its_load_arrived():
    ld = ["\t;;#ASMSTART", "\tglobal_load_dwordx4 v[10:13], v1, s[2:3] offset:0", "\t;;#ASMEND"]
    other = ["\t;;#ASMSTART", "\tglobal_load_dwordx4 v[20:23], v1, s[2:3] offset:1024", "\t;;#ASMEND"]
    ok = ld + other + ["s_waitcnt vmcnt(1)", "v_mov_b32_e32 v5, v10", "s_endpgm"]
    assert find_touched_before_arrival(ok) == (2, 0, [])
    early = ld + other + ["v_mov_b32_e32 v5, v10", "s_waitcnt vmcnt(1)", "s_endpgm"]
    assert len(find_touched_before_arrival(early)[2]) == 1
    third = ["\t;;#ASMSTART", "\tglobal_load_dwordx4 v[30:33], v1, s[2:3] offset:2048", "\t;;#ASMEND"]
    not_enough = ld + other + third + ["s_waitcnt vmcnt(3)", "v_mov_b32_e32 v5, v11", "s_waitcnt vmcnt(0)", "s_endpgm"]
    assert len(find_touched_before_arrival(not_enough)[2]) == 1
    # in flight across the barrier: a copy on the taken side of a branch, behind a loop's back edge, or to scratch memory
    for copy in ("v_mov_b32_e32 v5, v10", "v_accvgpr_write_b32 a7, v11", "scratch_store_dwordx4 off, v[10:13], off"):
        back = [".LBB0_1:", copy] + ld + ["s_barrier", "s_cbranch_scc1 .LBB0_1", "s_waitcnt vmcnt(0)", "s_endpgm"]
        side = ld + ["s_barrier", "s_cbranch_scc1 .LBB0_2", "s_waitcnt vmcnt(0)", "s_endpgm", ".LBB0_2:", copy, "s_endpgm"]
        late = ld + ["s_barrier", "s_waitcnt vmcnt(0)", "s_barrier", copy, "s_endpgm"]
        assert [len(find_touched_before_arrival(x)[2]) for x in (back, side, late)] == [1, 1, 0], copy
        assert find_touched_before_arrival(late)[:2] == (1, 1)


def test_lint_flags_a_late_writer():
    mf = ["\t;;#ASMSTART", "\tv_mfma_f32_16x16x32_bf16 a[0:3], v[90:93], v[54:57], a[0:3]", "\t;;#ASMEND"]
    assert len(find_late_writers(["v_accvgpr_write_b32 a1, 0"] + mf)[1]) == 1
    assert len(find_late_writers(["v_mov_b32_e32 v91, 0", "s_nop 1"] + mf)[1]) == 1
    assert find_late_writers(["v_accvgpr_write_b32 a1, 0", "s_nop 3"] + mf) == (1, [])
    assert find_late_writers(["v_accvgpr_write_b32 a9, 0"] + mf) == (1, [])
    assert find_late_writers(["v_accvgpr_write_b32 a1, 0", mf[1]]) == (0, [])   # not an asm MFMA: the compiler's job


def test_lint_flags_an_early_reader():
    ok = ["v_mfma_f32_16x16x32_bf16 v[2:5], v[90:93], v[50:53], v[2:5]",
          "v_mfma_f32_16x16x32_bf16 a[0:3], v[90:93], v[54:57], a[0:3]",
          "v_mfma_f32_16x16x32_bf16 a[4:7], v[90:93], v[58:61], a[4:7]",
          "v_mfma_f32_16x16x32_bf16 a[8:11], v[90:93], v[62:65], a[8:11]",
          "v_mov_b32_e32 v100, v2", "s_endpgm"]
    assert find_hazards(ok) == (1, [])
    assert find_hazards(ok, agpr_too=True)[0] == 4
    early = [ok[0], ok[1], "v_mov_b32_e32 v100, v2", "s_endpgm"]
    assert len(find_hazards(early)[1]) == 1
    via_branch = [ok[0], "s_cbranch_scc1 .LBB0_1", ok[1], ok[2], ok[3], "s_endpgm", ".LBB0_1:",
                  "v_add_f32_e32 v3, v3, v4", "s_endpgm"]
    assert len(find_hazards(via_branch)[1]) == 1
    in_place = [ok[0], ok[0], "s_endpgm"]          # accumulating into the same registers again is fine
    assert find_hazards(in_place) == (2, [])
    # an accumulator in the other register file read too early
    early_agpr = [ok[1], "v_accvgpr_read_b32 v7, a1", "s_endpgm"]
    assert find_hazards(early_agpr) == (0, [])
    assert len(find_hazards(early_agpr, agpr_too=True)[1]) == 1
    late_agpr = [ok[1], ok[2], ok[3], "v_accvgpr_read_b32 v7, a1", "s_endpgm"]
    assert find_hazards(late_agpr, agpr_too=True) == (3, [])


def test_no_hazard_around_the_mfmas_of_the_compiled_kernels(gemm_unit_asm):
    assert len(gemm_unit_asm) == 7
    for unit, lines in gemm_unit_asm.items():
        pinned, bad = find_hazards(lines, agpr_too=True)
        assert pinned > 0, f"{unit}: expected MFMAs"
        assert not bad, f"{unit}:\n" + "\n".join(bad[:10])
        n_asm, late = find_late_writers(lines)
        assert not late, f"{unit}:\n" + "\n".join(late[:10])
        stores = find_asm_stores(lines)
        assert not stores, f"{unit}: {len(stores)} stores\n" + "\n".join(stores[:10])
        n_loads, crossed, early = find_touched_before_arrival(lines)
        assert n_loads > 0 and crossed > 0 and not early, f"{unit}:\n" + "\n".join(early[:10])
