"""The contractions issue their MFMAs as inline asm, for which the compiler places no wait states (gfx950: a result of the 16x16x32 form
may be read 8 wait states after its issue, a vector instruction's result may be an operand 2 after it; it is what the compiler itself
leaves around its builtin).  The kernels wait by themselves, but copies of registers are the compiler's: every path of the listing is
walked from each MFMA, forwards for its result and backwards, through every branch that leads to it, for its operands."""
import os
import re
import subprocess

import pytest

from paper_2605_15609_amd import build as bld

RESULT, OPERAND = 8, 2


def _registers(text):
    out = set()
    for kind, lo, hi, one, n in re.findall(r"\b(?:([va])\[(\d+):(\d+)\]|([va])(\d+)\b)", text):
        out |= {(kind, i) for i in range(int(lo), int(hi) + 1)} if kind else {(one, int(n))}
    return out


def _listing(lines):
    """-> ([(opcode, operand text, registers per operand, written by hand)], {label: index})"""
    code, labels, by_hand = [], {}, False
    for line in lines:
        line = line.strip()
        if line.startswith((";;#ASMSTART", ";;#ASMEND")):
            by_hand = line.startswith(";;#ASMSTART")
        line = line.split(";")[0].strip()
        if line.endswith(":"):
            labels[line[:-1]] = len(code)
        elif line and line[0] not in ".#":
            op, _, args = line.partition(" ")
            code.append((op, args.strip(), [_registers(a) for a in re.split(r",(?![^\[]*\])", args)], by_hand))
    return code, labels


def _states(op, args):
    """wait states that an instruction stands for"""
    return int(args, 0) + 1 if op == "s_nop" else 1


def _predecessors(code, labels):
    before = [[] for _ in code]
    for i, (op, args, _, _) in enumerate(code):
        if op == "s_branch" or op.startswith("s_cbranch"):
            before[labels[args]].append(i)
        if op not in ("s_branch", "s_endpgm") and i + 1 < len(code):
            before[i + 1].append(i)
    return before


def _too_close(code, labels):
    bad, mfmas = [], 0
    before = _predecessors(code, labels)
    for i, (op, args, regs, by_hand) in enumerate(code):
        if not (by_hand and op.startswith("v_mfma")):
            continue
        mfmas += 1
        operands = set().union(*regs[1:])
        todo, seen = [(j, 0) for j in before[i]], {}
        while todo:
            j, waited = todo.pop()
            if waited >= OPERAND or seen.get(j, OPERAND) <= waited:
                continue
            seen[j] = waited
            o, a, r, _ = code[j]
            written = r[0] | r[1] if "swap" in o else r[0]
            if o.startswith("v_") and not o.startswith("v_mfma") and written & operands:
                bad.append((o, a, args, waited))
            todo += [(k, waited + _states(o, a)) for k in before[j]]
        todo, seen = [(i + 1, 0)], {}
        while todo:
            j, waited = todo.pop()
            if waited >= RESULT or seen.get(j, RESULT) <= waited:
                continue
            seen[j] = waited
            o, a, r, _ = code[j]
            if o.startswith("v_mfma"):      # (the same accumulators again need no wait)
                todo.append((j + 1, waited + 1))
            elif o.startswith(("v_", "ds_", "buffer_", "global_", "scratch_")) and regs[0] & set().union(*r):
                bad.append((args, o, a, waited))
            elif o != "s_endpgm":
                if o == "s_branch" or o.startswith("s_cbranch"):
                    todo.append((labels[a], waited + 1))
                if o != "s_branch":
                    todo.append((j + 1, waited + _states(o, a)))
    return bad, mfmas


MFMA = ";;#ASMSTART\nv_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]\n;;#ASMEND\n"


@pytest.mark.parametrize("listing,close", [
    ("v_mov_b32_e32 v4, v9\n" + MFMA, 1),
    ("v_mov_b32_e32 v4, v9\ns_nop 0\n" + MFMA, 1),
    ("v_mov_b32_e32 v4, v9\ns_nop 1\n" + MFMA, 0),
    ("v_mov_b32_e32 v8, v9\n" + MFMA, 0),
    ("v_permlane32_swap_b32_e32 v8, v4\n" + MFMA, 1),
    (".LBB0_1:\n" + MFMA + "s_nop 7\nv_mov_b32_e32 v4, v9\ns_cbranch_scc1 .LBB0_1\n", 1),                 # a copy at the loop's end
    ("s_branch .LBB0_2\nv_mov_b32_e32 v4, v9\n.LBB0_2:\n" + MFMA, 1),                                      # (by falling through)
    ("v_mov_b32_e32 v4, v9\ns_branch .LBB0_3\n.LBB0_2:\n" + MFMA + "s_endpgm\n.LBB0_3:\ns_branch .LBB0_2\n", 0),
    (MFMA + "s_nop 6\nv_accvgpr_read_b32 v9, a1\n", 1),
    (MFMA + "s_nop 7\nv_accvgpr_read_b32 v9, a1\n", 0),
])
def test_the_walk(listing, close):
    bad, mfmas = _too_close(*_listing((listing + "s_endpgm\n").splitlines()))
    assert mfmas == 1 and len(bad) == close, bad


@pytest.mark.parametrize("source", ["gemm_mfma.hip", "lm_head.hip"])
def test_wait_states_around_hand_written_mfmas(source, tmp_path):
    out = str(tmp_path / "listing.s")
    subprocess.run([bld._hipcc(), *bld.FLAGS, "--cuda-device-only", "-S", os.path.join(bld.CSRC, source), "-o", out], check=True, capture_output=True)
    bad, mfmas = _too_close(*_listing(open(out)))
    assert mfmas > 100 and not bad, bad[:4]
