"""Matrix instructions of gfx950 have no interlock for a vector or memory instruction that reads (or overwrites) their result
too early: the compiler counts the instructions in between and fills up with s_nop.  ROCm 7.2 has left such a gap on the path
of a branch that skips code between the two (an aggregated state came out wrong), and whether it does depends on how a kernel
happens to be laid out.  So the code that was built is walked here: every kernel of the library, disassembled, from every
matrix instruction along every path of its control flow to the first readers and writers of its result.

The same goes for a scalar register that a vector instruction writes (v_readfirstlane, v_readlane of a spilled one, a
comparison) and a memory instruction reads: five wait states, which the compiler keeps for its own memory instructions, not for
one that stands in inline assembly (k_ffn_fused.hip's loads into LDS), since it doesn't see what that one reads."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2205_14756_amd import build as msla_build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"

# Wait states from a matrix instruction to another kind of instruction that touches its result, as the compiler keeps them on
# gfx950: 16-bit inputs, passes + 3, one more above two passes (4x4x4: 2 passes, 16x16: 4, 32x32x16: 8); fp32 inputs, passes + 2
# (16x16x4: 8).
NEED = {"4x4x4_16b": 5, "16x16x16": 8, "16x16x32": 8, "32x32x16": 12, "16x16x4_f32": 10}


def need(op):
    found = [n for k, n in NEED.items() if k in op]
    assert len(found) == 1, f"a matrix instruction that is not in the table: {op}"
    return found[0]


def registers(text):
    out = set()
    for m in re.finditer(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)", text):
        kind, a = m.group(1), int(m.group(2) or m.group(4))
        out.update((kind, i) for i in range(a, int(m.group(3) or a) + 1))
    return out


def kernels(listing):
    """{name: [(operation, operands, index of a branch's target or None)]} of an objdump listing"""
    out = {}
    for part in re.split(r"^[0-9a-f]+ <", listing, flags=re.M)[1:]:
        name, body = part.split(">:", 1)
        rows = re.findall(r"^\t(\S+)[ \t]*([^\n]*?)[ \t]*// ([0-9A-F]+):[^\n]*?(?:<[^\n>]*?\+0x([0-9a-f]+)>)?$", body, flags=re.M)
        if not rows:
            continue
        start = int(rows[0][2], 16)
        at = {int(r[2], 16) - start: i for i, r in enumerate(rows)}
        out[name] = [(op, args, at[int(t, 16)] if t and op.startswith(("s_branch", "s_cbranch")) else None)
                     for op, args, _, t in rows]
    return out


def gaps(code):
    """[(matrix instruction's index, reader's index, wait states, wait states needed)] of results that are touched too early"""
    bad = []
    for i, (op, args, _) in enumerate(code):
        if not op.startswith("v_mfma"):
            continue
        wanted, result = need(op), registers(args.split(",")[0])
        seen, todo = {}, [(i + 1, 0)]
        while todo:
            j, waited = todo.pop()
            if j >= len(code) or waited >= wanted or seen.get(j, wanted) <= waited:
                continue
            seen[j] = waited
            o, a, target = code[j]
            if o == "s_endpgm":
                continue
            if o.startswith("v_mfma"):
                # (another matrix instruction: its addend may be the result at once, its factors may not)
                parts = re.split(r",(?![^\[]*\])", a)
                if result & (registers(parts[1]) | registers(parts[2])):
                    bad.append((i, j, waited, wanted))
                    continue
                if result <= registers(parts[0]):
                    continue                            # it takes the result over
            elif o.startswith(("v_", "buffer_", "global_", "flat_", "scratch_", "ds_")) and result & registers(a):
                bad.append((i, j, waited, wanted))
                continue
            if target is not None:
                todo.append((target, waited + 1))
            if o != "s_branch":
                todo.append((j + 1, waited + (int(a) + 1 if o == "s_nop" else 1)))
    return bad


SGPR_TO_MEMORY = 5          # wait states from a vector instruction's write of a scalar register to a memory instruction's read
MEMORY = ("buffer_", "global_", "flat_", "scratch_")


def scalars(text):
    out = set(re.findall(r"\b(vcc|m0)\b", text))
    for m in re.finditer(r"\bs(?:\[(\d+):(\d+)\]|(\d+)\b)", text):
        a = int(m.group(1) or m.group(3))
        out.update(range(a, int(m.group(2) or a) + 1))
    return out


def scalar_results(op, args):
    """scalar registers that a vector instruction writes: its first operand, or its second (the carry) behind a vector register"""
    parts = re.split(r",(?![^\[]*\])", args)
    wide = ("v_add_co", "v_addc_co", "v_sub_co", "v_subb_co", "v_subrev_co", "v_subbrev_co", "v_div_scale", "v_mad_u64_u32", "v_mad_i64_i32")
    return scalars(parts[1] if op.startswith(wide) else parts[0])


def early_scalar_reads(code):
    """[(writer's index, memory instruction's index, wait states)] of scalar registers that are read too early"""
    bad = []
    for i, (op, args, _) in enumerate(code):
        written = scalar_results(op, args) if op.startswith("v_") else set()
        if not written:
            continue
        seen, todo = {}, [(i + 1, 0)]
        while todo:
            j, waited = todo.pop()
            if j >= len(code) or waited >= SGPR_TO_MEMORY or seen.get(j, SGPR_TO_MEMORY) <= waited:
                continue
            seen[j] = waited
            o, a, target = code[j]
            if o.startswith(MEMORY) and written & (scalars(a) | ({"m0"} if a.endswith(" lds") else set())):
                bad.append((i, j, waited))
                continue
            if o == "s_endpgm":
                continue
            if target is not None:
                todo.append((target, waited + 1))
            if o != "s_branch":
                todo.append((j + 1, waited + (int(a) + 1 if o == "s_nop" else 1)))
    return bad


def unguarded_lds_loads(code):
    """indexes of loads straight into LDS that don't have, whatever the compiler put there, five wait states right before them (of s_nop, moves
    of m0 and loads before them), and one of s_nop behind a move of m0"""
    bad = []
    for i, (op, args, _) in enumerate(code):
        if not (op.startswith("buffer_load") and args.endswith(" lds")):
            continue
        j, waited = i - 1, 0
        while j >= 0 and (code[j][0] == "s_nop" or (code[j][1].endswith(" lds") and waited) or
                          (code[j][0].startswith("s_") and code[j][1].startswith("m0,") and waited)):
            waited += int(code[j][1]) + 1 if code[j][0] == "s_nop" else 1
            j -= 1
        # (a branch to the load itself would go round them)
        if waited < SGPR_TO_MEMORY or any(t is not None and j + 1 < t <= i for _, _, t in code):
            bad.append(i)
    return bad


def built_kernels(tmp_path):
    if not os.path.exists(msla_build.LIB):
        msla_build.build(True)
    lib = shutil.copy(msla_build.LIB, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=tmp_path, check=True, capture_output=True, timeout=300)
    objects = sorted(f for f in os.listdir(tmp_path) if f.endswith("gfx950"))
    assert objects, "no device code in the library"
    for f in objects:
        listing = subprocess.run([OBJDUMP, "-d", f], cwd=tmp_path, check=True, capture_output=True, text=True, timeout=300).stdout
        yield from kernels(listing).items()


def test_the_walk_finds_a_gap_behind_a_branch():
    # six wait states on the straight path; the branch jumps over four of them
    text = """
0000000000001000 <k>:
	v_mfma_f32_4x4x4_16b_f16 v[0:3], v[8:9], v[10:11], v[0:3]  // 000000001000: 00000000
	s_cbranch_scc1 3                                           // 000000001008: BF850003 <k+0x18>
	s_nop 3                                                    // 00000000100C: BF800003
	s_mov_b32 s0, 0                                            // 000000001010: BE800080
	s_mov_b32 s1, 0                                            // 000000001014: BE800080
	v_cvt_f16_f32_e32 v4, v2                                   // 000000001018: 00000000
	s_endpgm                                                   // 00000000101C: BF810000
"""
    (code,) = kernels(text).values()
    assert gaps(code) == [(0, 5, 1, 5)]
    code[1] = ("s_nop", "0", None)
    assert gaps(code) == []


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="needs the ROCm toolchain's objdump")
def test_every_matrix_result_of_the_built_library_is_waited_for(tmp_path):
    seen, bad = 0, []
    for name, code in built_kernels(tmp_path):
        n = sum(op.startswith("v_mfma") for op, _, _ in code)
        seen += n
        bad += [f"{name}: {code[i]} -> {code[j]} after {w} of {need_} wait states" for i, j, w, need_ in gaps(code)]
    assert seen > 1000, f"only {seen} matrix instructions were found: the listing is read wrongly"
    assert not bad, "\n".join(bad[:20])


def test_the_walk_finds_an_early_read_of_a_scalar_register():
    text = """
0000000000001000 <k>:
	v_readfirstlane_b32 s5, v1                                 // 000000001000: 00000000
	s_cbranch_scc1 2                                           // 000000001004: BF850002 <k+0x10>
	s_nop 3                                                    // 000000001008: BF800003
	s_mov_b32 m0, s0                                           // 00000000100C: BE800080
	s_nop 0                                                    // 000000001010: BF800000
	buffer_load_dwordx4 v2, s[4:7], 0 offen lds                // 000000001014: 00000000
	v_cmp_gt_u32_e64 s[8:9], v0, v1                            // 00000000101C: 00000000
	global_load_dword v3, v2, s[8:9]                           // 000000001024: 00000000
	v_add_co_u32_e64 v4, s[10:11], s12, v0                     // 00000000102C: 00000000
	buffer_load_dword v5, v2, s[12:15], 0 offen                // 000000001034: 00000000
	s_endpgm                                                   // 00000000103C: BF810000
"""
    (code,) = kernels(text).values()
    # s5 through the branch, and the comparison's pair; s[12:15] was not written by the addition
    assert early_scalar_reads(code) == [(0, 5, 2), (6, 7, 0)]
    assert unguarded_lds_loads(code) == [5]
    # (a second load rests on the first one's wait; none of them may follow a move of m0 at once)
    pair = [("s_nop", "4", None), code[5], ("s_add_u32", "m0, m0, 0x1000", None), ("s_nop", "0", None), code[5]]
    assert unguarded_lds_loads(pair) == [] and unguarded_lds_loads(pair[:3] + pair[4:]) == [3] and unguarded_lds_loads(pair[1:]) == [0, 3]
    code[1], code[4] = ("s_nop", "0", None), ("s_nop", "4", None)
    assert early_scalar_reads(code) == [(6, 7, 0)]
    assert unguarded_lds_loads(code) == []


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="needs the ROCm toolchain's objdump")
def test_scalar_registers_reach_memory_instructions_in_time(tmp_path):
    loads, bad = 0, []
    for name, code in built_kernels(tmp_path):
        loads += sum(op.startswith("buffer_load") and args.endswith(" lds") for op, args, _ in code)
        bad += [f"{name}: {code[i]} -> {code[j]} after {w} of {SGPR_TO_MEMORY} wait states" for i, j, w in early_scalar_reads(code)]
        bad += [f"{name}: {code[i]} relies on what the compiler put before it" for i in unguarded_lds_loads(code)]
    assert loads > 50, f"only {loads} loads into LDS were found: the listing is read wrongly"
    assert not bad, f"{len(bad)}:\n" + "\n".join(bad[:20])
