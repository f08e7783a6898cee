"""The contractions issue their MFMAs as inline asm, for which the compiler places no wait states (gfx950: a result of the 16x16x32 form
may be read 8 wait states after its issue, a vector instruction's result may be an operand 2 after it; it is what the compiler itself
leaves around its builtin).  The kernels wait by themselves, but copies of registers are the compiler's: every path of the listing is
walked from each MFMA."""
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


def _listing(path):
    """-> ([(opcode, operand text, registers per operand, written by hand)], {label: index})"""
    code, labels, by_hand = [], {}, False
    for line in open(path):
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


def _too_close(code, labels):
    bad, mfmas = [], 0
    for i, (op, args, regs, by_hand) in enumerate(code):
        if not (by_hand and op.startswith("v_mfma")):
            continue
        mfmas += 1
        for back in range(1, OPERAND + 1):
            o, _, r, _ = code[i - back]
            if o == "s_nop":
                break
            if o.startswith("v_") and not o.startswith("v_mfma") and r[0] & set().union(*regs[1:]):
                bad.append((code[i - back], args))
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
                    todo.append((j + 1, waited + (int(a) + 1 if o == "s_nop" else 1)))
    return bad, mfmas


@pytest.mark.parametrize("source", ["gemm_mfma.hip", "lm_head.hip"])
def test_wait_states_around_hand_written_mfmas(source, tmp_path):
    out = str(tmp_path / "listing.s")
    subprocess.run([bld._hipcc(), *bld.FLAGS, "--cuda-device-only", "-S", os.path.join(bld.CSRC, source), "-o", out], check=True, capture_output=True)
    bad, mfmas = _too_close(*_listing(out))
    assert mfmas > 100 and not bad, bad[:4]
