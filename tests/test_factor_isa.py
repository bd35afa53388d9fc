"""The leaf factorization of factor.hip broadcasts doubles through DPP operands in inline assembly, whose hazards the compiler
does not see: a DPP operand must not have been written by a vector instruction less than two wait states before (an
instruction is one, s_nop n is n + 1), nor any operand by a transcendental one directly before.  The statements keep
these distances as long as the compiler places no copy of an operand right in front of one.  This test compiles the
file the way the build does and checks every such instruction in the generated ISA (CPU only)."""
import os
import re
import shutil
import subprocess

import pytest

DPP_WAIT, TRANS_WAIT = 2, 1


def _regs(op):
    """Vector registers of an operand: v5, v[4:5], -v[4:5], |v3|."""
    m = re.search(r"\bv\[(\d+):(\d+)\]", op)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    m = re.search(r"\bv(\d+)\b", op)
    return {int(m.group(1))} if m else set()


def _instructions(text):
    """(mnemonic, operands) per instruction; (None, []) for a label."""
    out = []
    for line in text.split("\n"):
        if re.match(r"^[.\w$]+:", line):
            out.append((None, []))
            continue
        m = re.match(r"\s+([vs]_\w+|ds_\w+|buffer_\w+|global_\w+|scratch_\w+|flat_\w+)\s*([^;]*)", line)
        if m:
            out.append((m.group(1), [o.strip() for o in m.group(2).split(",")]))
    return out


def violations(text):
    """(number of 64-bit DPP instructions, those that follow a write of an operand too closely)."""
    ins, n, bad = _instructions(text), 0, []
    for i, (op, args) in enumerate(ins):
        if op is None or not re.fullmatch(r"v_\w*64\w*_dpp", op):
            continue
        n += 1
        src = [_regs(a.split(" ")[0]) for a in args[1:]]
        used = set().union(*src) | (_regs(args[0]) if "fmac" in op else set())
        states, k = 0, i - 1
        while k >= 0 and states < DPP_WAIT:
            p, pargs = ins[k]
            if p is None:
                bad.append((i, "a label closer than the distance"))
                break
            if p == "s_nop":
                states += int(pargs[0]) + 1
            else:
                if p.startswith("v_") and not p.startswith("v_cmp"):
                    written = _regs(pargs[0])
                    if written & src[0]:
                        bad.append((i, f"{p} {', '.join(pargs)} before {op} {', '.join(args)}"))
                        break
                    if states < TRANS_WAIT and re.match(r"v_(rcp|rsq|sqrt|exp|log|sin|cos)_", p) and written & used:
                        bad.append((i, f"{p} {', '.join(pargs)} before {op} {', '.join(args)}"))
                        break
                states += 1
            k -= 1
    return n, bad


@pytest.mark.parametrize("between,ok", [
    ("", False), ("\ts_nop 0\n", False), ("\tv_mov_b32_e32 v9, v8\n", False), ("\ts_nop 1\n", True),
    ("\tv_mov_b32_e32 v9, v8\n\ts_nop 0\n", True), ("\ts_nop 1\n.LBB0_1:\n", False),
])
def test_checker_sees_short_distances(between, ok):
    dpp = "\tv_fmac_f64_dpp v[2:3], v[4:5], v[6:7] row_newbcast:1 row_mask:0xf bank_mask:0xf\n"
    n, bad = violations("\tv_mov_b32_e32 v5, v1\n" + between + dpp)
    assert n == 1 and (not bad) == ok
    assert violations("\tv_rcp_f64_e32 v[6:7], v[0:1]\n" + dpp)[1]            # a transcendental result, used at once
    assert not violations("\tv_mov_b32_e32 v6, v1\n" * 2 + dpp)[1]            # a plain one in the operand that is not DPP


def test_dpp_operands_keep_their_distance(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    from paper_2603_28845_amd import build
    out = tmp_path / "factor.s"
    cmd = [hipcc, *build.HIPCC_FLAGS, *build.EXTRA_FLAGS.get("factor.hip", []), "-S", "--cuda-device-only",
           os.path.join(build.CSRC, "factor.hip"), "-o", str(out)]
    subprocess.run(cmd, check=True, capture_output=True)
    n, bad = violations(out.read_text())
    # a leaf: 16 broadcasts of a pivot, 120 updates and 36 eliminations; it is inlined four times (two kernels, the first
    # leaf and the others)
    assert n == 4 * (16 + 120 + 36)
    assert not bad, bad[:5]
