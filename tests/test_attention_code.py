"""What the compiler makes of the attention kernels.  Over key ranges the scores' multiplies are inline assembly that its hazard rules do not
see: every other use of a score is far enough behind the multiply, and no register goes to memory in the loops.  In the fp32 tile kernel the
output products go beside the softmax."""
import os
import re
import subprocess

import pytest

from paper_2505_21467_amd import build

MULTIPLY = 4   # wait states (of four clocks) that a 16x16x32 multiply keeps the matrix core
NEEDED = 20    # between a multiply and the first use of its result by anything but the multiply that adds to it: twice what its four passes ask for


def _registers(text):
    """Numbers of the VALU's registers that an operand names."""
    out = set()
    for a, b, c in re.findall(r"\bv(?:\[(\d+):(\d+)\]|(\d+)\b)", text):
        out.update(range(int(a), int(b) + 1) if a else [int(c)])
    return out


def _kernels(asm, kernel):
    """(name, instructions, place of each label, bytes of scratch) of every instance of a kernel; an instruction: (opcode, operands, in inline assembly)."""
    lines, out = asm.split("\n"), []
    for start, line in enumerate(lines):
        if not re.match(r"_Z\S*%s\S*:" % kernel, line):
            continue
        code, labels, inline = [], {}, False
        for at in range(start + 1, len(lines)):
            text = lines[at].split(";")[0].strip() if not lines[at].strip().startswith(";;#") else lines[at].strip()
            if text.startswith(";;#"):
                inline = "ASMSTART" in text
            elif text.startswith(".Lfunc_end"):
                break
            elif text.endswith(":"):
                labels[text[:-1]] = len(code)
            elif text and not text.startswith("."):
                op, _, rest = text.partition(" ") if "\t" not in text else text.partition("\t")
                code.append((op, rest.strip(), inline))
        scratch = next(int(m.group(1)) for m in (re.match(r"; ScratchSize: (\d+)", l) for l in lines[at:]) if m)
        out.append((line.split(":")[0], code, labels, scratch))
    return out


def _nearest_use(code, labels, at):
    """Wait states between the multiply at `at` and the first other use of its result, NEEDED or more if there is none nearer."""
    result = _registers(code[at][1].split(",")[0])
    todo, seen, nearest = [(at + 1, 0)], {}, NEEDED
    while todo:
        i, far = todo.pop()
        while i < len(code) and far < nearest and seen.get(i, NEEDED) > far:
            seen[i] = far
            op, rest, _ = code[i]
            operands = [_registers(x) for x in re.split(r",\s*(?![^\[]*\])", rest)]
            if op.startswith("v_mfma"):
                d, a, b, c = (operands + [set()] * 4)[:4]
                if result & (a | b) or any(x & result and x != result for x in (d, c)):
                    nearest = far
                if d == result:
                    break  # (the next multiply of the sum, which has its own distance)
                far += MULTIPLY
            else:
                if any(x & result for x in operands):
                    nearest = far
                far += int(rest, 0) + 1 if op == "s_nop" else 1
            if op.startswith("s_cbranch") or op == "s_branch":
                todo.append((labels[rest], far))
            if op in ("s_branch", "s_endpgm"):
                break
            i += 1
    return nearest


def _compiled(folder, source):
    out = str(folder.mktemp("asm") / "code.s")
    cmd = [build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, source), "-o", out]
    subprocess.run(cmd, check=True, capture_output=True, timeout=240)
    with open(out) as f:
        return f.read()


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    found = _kernels(_compiled(tmp_path_factory, "fc_attn_mfma.hip"), "k_attn_ranges")
    assert len(found) == 10
    return found


def test_scores_are_used_far_enough_behind_their_multiplies(kernels):
    for name, code, labels, _ in kernels:
        multiplies = [i for i, (op, _, inline) in enumerate(code) if inline and op.startswith("v_mfma")]
        assert len(multiplies) >= 32, name
        for i in multiplies:
            far = _nearest_use(code, labels, i)
            assert far >= NEEDED, "%s: %s used after %d wait states" % (name, code[i], far)


def test_no_register_goes_to_memory(kernels):
    """(A reload in the loop waits for the keys and values under way as well: the ring would hold nothing ahead.)"""
    for name, code, _, scratch in kernels:
        assert scratch == 0 and not any(op.startswith("scratch_") for op, _, _ in code), (name, scratch)


def test_a_use_too_near_is_found():
    """The check itself: a read behind one, two and four other multiplies, by way of a branch, and of another register."""
    other = ("v_mfma_f32_16x16x32_bf16", "v[8:11], v[40:43], v[44:47], 0", True)

    def far(*rest):
        code = [("v_mfma_f32_16x16x32_bf16", "v[0:3], v[40:43], v[44:47], 0", True), *rest, ("s_endpgm", "", False)]
        return _nearest_use(code, {".LBB0_1": len(code) - 2}, 0)

    read = ("v_fma_f32", "v20, s3, v2, v21", False)
    assert far(read) == 0 and far(other, read) == 4 and far(other, other, read) == 8 and far(*5 * [other], read) == NEEDED
    assert far(("s_cbranch_vccnz", ".LBB0_1", False), ("s_nop", "15", False), read) == 1
    assert far(("s_nop", "15", False), ("s_nop", "3", False), read) == NEEDED and far(("v_fma_f32", "v20, s3, v4, v21", False)) == NEEDED
    assert far(("v_mfma_f32_16x16x32_bf16", "v[0:3], v[40:43], v[44:47], v[0:3]", True), read) == NEEDED


def test_fp32_tile_products_go_beside_the_softmax(tmp_path_factory):
    """The loop over whole groups has a group's exponentials (nine per tile of 16 rows) and its output products without a branch between them
    (those for halves of groups, there, took up to 6 % of a call)."""
    found = _kernels(_compiled(tmp_path_factory, "fc_generic.hip"), r"k_attn_tileIfLi\d+ELi\d+ELi\d+ELb1E")
    assert len(found) == 7
    for name, code, labels, scratch in found:
        tiles = int(re.search(r"k_attn_tileIfLi\d+ELi(\d+)E", name).group(1))
        starts = set(labels.values()) | {i + 1 for i, (op, _, _) in enumerate(code) if op.startswith("s_cbranch")}
        edges = sorted(starts | {0, len(code)})
        both = 0
        for a, b in zip(edges, edges[1:]):
            ops = [op for op, _, _ in code[a:b]]
            if any(op.startswith("v_mfma") for op in ops):
                both += sum(op.startswith("v_exp") for op in ops)
        assert both >= 9 * tiles and scratch == 0, (name, both)
