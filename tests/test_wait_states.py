"""Matrix instructions of gfx950 have no interlock for a vector or memory instruction that reads (or overwrites) their result
too early: the compiler counts the instructions in between and fills up with s_nop.  ROCm 7.2 has left such a gap on the path
of a branch that skips code between the two (an aggregated state came out wrong), and whether it does depends on how a kernel
happens to be laid out.  So the code that was built is walked here: every kernel of the library, disassembled, from every
matrix instruction along every path of its control flow to the first readers and writers of its result."""
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
    if not os.path.exists(msla_build.LIB):
        msla_build.build(True)
    lib = shutil.copy(msla_build.LIB, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=tmp_path, check=True, capture_output=True, timeout=300)
    objects = sorted(f for f in os.listdir(tmp_path) if f.endswith("gfx950"))
    assert objects, "no device code in the library"
    seen, bad = 0, []
    for f in objects:
        listing = subprocess.run([OBJDUMP, "-d", f], cwd=tmp_path, check=True, capture_output=True, text=True, timeout=300).stdout
        for name, code in kernels(listing).items():
            n = sum(op.startswith("v_mfma") for op, _, _ in code)
            seen += n
            bad += [f"{name}: {code[i]} -> {code[j]} after {w} of {need_} wait states" for i, j, w, need_ in gaps(code)]
    assert seen > 1000, f"only {seen} matrix instructions were found: the listing is read wrongly"
    assert not bad, "\n".join(bad[:20])
