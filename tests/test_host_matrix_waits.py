"""A matrix instruction's result may not be touched by another instruction for some wait
states, which the compiler has to put there. Checked on the built instructions of the bf16
family, along every path through a kernel: an accumulator read too early would be stale,
and only in some lanes and runs."""
import re

import codeobj
from paper_2008_03602_amd import _lib as L

# wait states between the instruction and the first other one that reads or writes its
# result, on gfx950: its passes of 4 clocks, plus 4
WAITS = {"v_mfma_f32_16x16x32_bf16": 4 + 4, "v_mfma_f32_32x32x16_bf16": 8 + 4}


def _registers(text):
    out = set()
    for m in re.finditer(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)", text):
        lo = int(m.group(2) or m.group(4))
        out |= {(m.group(1), i) for i in range(lo, int(m.group(3) or lo) + 1)}
    return out


def _early_touches(rows, at):
    """Instructions that touch the result of matrix instruction `at` within its wait."""
    need, operands = WAITS[rows[at][1]], rows[at][2].split(", ")
    result = _registers(operands[0])
    index = {r[0]: i for i, r in enumerate(rows)}
    best, todo = {}, [(at + 1, 0)]
    while todo:
        i, waited = todo.pop()
        if i >= len(rows) or waited >= need or best.get(i, need) <= waited:
            continue
        best[i] = waited
        _, op, args, target = rows[i]
        if op == "s_endpgm":
            continue
        if op.startswith("s_cbranch") or op == "s_branch":
            todo.append((index[target], waited + 1))
            if op == "s_branch":
                continue
        if op.startswith("v_mfma"):
            o = args.split(", ")
            if _registers(o[0]) == result and _registers(o[3]) == result:
                continue  # accumulates on: forwarded, and a result of its own
        if not op.startswith("s_") and _registers(args) & result:
            yield waited, op, args
            continue
        todo.append((i + 1, waited + (int(args, 0) if op == "s_nop" else 0) + 1))


def test_matrix_results_are_left_alone_for_their_wait():
    kernels = checked = 0
    for sym, rows in codeobj.instructions(L.LIB_PATH, "igemm_bf16_kernel"):
        kernels += 1
        for i, r in enumerate(rows):
            if r[1].startswith("v_mfma"):
                checked += 1
                early = list(_early_touches(rows, i))
                assert not early, (sym, hex(r[0]), r[1], early)
    assert kernels >= 90 and checked >= 10 * kernels


def test_the_check_sees_an_early_copy():
    # a loop that ends in a copy of the result: too early after the last product on the
    # way out, and late enough behind 8 wait states
    def rows(nop):
        return [(0, "v_mfma_f32_16x16x32_bf16", "v[0:3], v[4:7], v[8:11], v[0:3]", None),
                (8, "s_cbranch_scc1", "65533", 0),
                (12, "s_nop", nop, None),
                (16, "v_mov_b32_e32", "v20, v2", None),
                (20, "s_endpgm", "", None)]
    assert [e[1] for e in _early_touches(rows("5"), 0)] == ["v_mov_b32_e32"]
    assert not list(_early_touches(rows("6"), 0))
