"""Properties of the Gram kernels that only the generated code shows.  These tests compile gram.hip the way the build does
and look at the ISA (CPU only).

The 384 x 256 kernel pins its accumulator tiles through inline-assembly MFMAs, which the compiler's hazard handling
cannot see: the loop is only correct while the compiler neither spills nor copies an accumulator inside it.

The fp32 and bf16 kernels whose waves share out the tokens take what lies behind a run's last token as zero, from the
bounds check of their buffer loads.  An instruction's scalar offset is no part of that check, so only batches that lie inside the run may
use one."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _isa(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    from paper_2603_28845_amd import build
    out = tmp_path / "gram.s"
    cmd = [hipcc, *build.HIPCC_FLAGS, *build.EXTRA_FLAGS.get("gram.hip", []), "-S", "--cuda-device-only",
           os.path.join(build.CSRC, "gram.hip"), "-o", str(out)]
    subprocess.run(cmd, check=True, capture_output=True)
    return out.read_text()


def test_wide_gram_loop_is_straight_line(tmp_path):
    text = _isa(tmp_path)
    found = 0
    for m in re.finditer(r"^(_ZN\S*gram_bf16_ring_kernelINS\d+_8RingWideELb[01]E\S*):[^\n]*\n(.*?)^\.Lfunc_end", text, re.S | re.M):
        body = m.group(2).split("\n")
        mf = [i for i, l in enumerate(body) if "v_mfma_f32_32x32x16_bf16" in l]
        assert len(mf) == 48, (m.group(1), len(mf))           # two half-iterations of 24 tiles, nowhere else
        loop = body[mf[0]:mf[-1] + 1]
        assert not any("scratch_" in l for l in loop), "an accumulator or operand is spilled inside the loop"
        assert not any("v_accvgpr" in l for l in loop), "an accumulator is copied between the register halves inside the loop"
        acc = set()
        for i in mf:                                          # 16 tiles in AGPRs, 8 in VGPRs, each its own registers
            acc.add(re.search(r"v_mfma_f32_32x32x16_bf16 ([av]\[\d+:\d+\])", body[i]).group(1))
        assert len(acc) == 24 and sum(a.startswith("a[") for a in acc) == 16
        # the last MFMA of the loop body carries its own wait states, inside the same assembly statement, so that
        # whatever the compiler places at the loop's exit reads retired accumulators
        assert [l.strip() for l in body[mf[-1] + 1:mf[-1] + 4]] == ["s_nop 15", "s_nop 15", ";;#ASMEND"], \
            "no wait states after the last MFMA of the loop"
        found += 1
    assert found == 3        # the symmetric kernel, its paced form and the cross kernel


def test_paced_gram_loop_is_placed(tmp_path):
    """The paced loop's place in the 32-byte windows of the instruction fetch is 4 % of the widest calls: 24 or 28 bytes into one."""
    hipcc, objdump = shutil.which("hipcc") or "/opt/rocm/bin/hipcc", "/opt/rocm/llvm/bin/llvm-objdump"
    if not os.path.exists(hipcc) or not os.path.exists(objdump):
        pytest.skip("no hipcc or llvm-objdump")
    from paper_2603_28845_amd import build
    out = tmp_path / "gram.co"
    subprocess.run([hipcc, *build.HIPCC_FLAGS, *build.EXTRA_FLAGS.get("gram.hip", []), "-c", "--cuda-device-only", "--no-gpu-bundle-output",
                    os.path.join(build.CSRC, "gram.hip"), "-o", str(out)], check=True, capture_output=True)
    text = subprocess.run([objdump, "-d", "--no-show-raw-insn", str(out)], check=True, capture_output=True, text=True).stdout
    body = re.search(r"^[0-9a-f]+ <\S*gram_bf16_ring_kernelINS\d+_8RingWideELb0ELb1E\S*>:\n(.*?)^\n", text + "\n", re.S | re.M).group(1)
    ins = [(int(m.group(2), 16), m.group(1)) for m in re.finditer(r"^\s+(.*?)\s*// ([0-9A-F]+):", body, re.M)]
    first, last = [a for a, i in ins if i.startswith("v_mfma")][::47]
    starts = set()
    for a, i in ins:
        m = re.match(r"s_cbranch\S* (\d+)", i)
        if m and a > last:
            to = a + 4 + 4 * (int(m.group(1)) - (65536 if int(m.group(1)) >= 32768 else 0))
            if first - 512 < to <= first:
                starts.add(to)
    assert len(starts) == 1 and starts.pop() % 32 in (24, 28)


@pytest.fixture(scope="module")
def isa(tmp_path_factory):
    return _isa(tmp_path_factory.mktemp("isa"))


@pytest.mark.parametrize("mt,steps", [(1, 16), (2, 8)])   # 32 x 32 tiles per side, loads of a batch per operand tile
def test_f32_runs_check_every_offset_past_the_run(isa, mt, steps):
    body = re.search(r"^_ZN\S*gram_f32_split_kernelILi%dE\S*:[^\n]*\n(.*?)^\.Lfunc_end" % mt, isa, re.S | re.M).group(1)
    loads = [m.group(1) for m in re.finditer(r"buffer_load_dword v\d+, v\d+, s\[\d+:\d+\], (\S+) offen", body)]
    operands = mt + 2 * mt                                    # diagonal tiles load one operand, the others two
    # per kind of tile: the first batch, two batches inside the run, two that may reach past its end
    assert len(loads) == 5 * steps * operands
    # the first pair of tokens of a batch has offset 0; every other load of the two inside batches has a scalar offset
    assert sum(o != "0" for o in loads) == 2 * (steps - 1) * operands
    # kinds of tile one after the other: the first batch and the last two of each carry no scalar offset
    sizes = sorted((mt, 2 * mt), reverse=loads.index(next(o for o in loads if o != "0")) > steps * mt + mt)
    pos = 0
    for per_step in sizes:
        n = steps * per_step
        first, inside, past = loads[pos:pos + n], loads[pos + n:pos + 3 * n], loads[pos + 3 * n:pos + 5 * n]
        assert all(o == "0" for o in first) and all(o == "0" for o in past)
        assert sum(o != "0" for o in inside) == 2 * (steps - 1) * per_step
        pos += 5 * n
    assert pos == len(loads)


def test_bf16_runs_check_every_offset_past_the_run(isa):
    body = re.search(r"^_ZN\S*gram_bf16_split_kernel\S*:[^\n]*\n(.*?)^\.Lfunc_end", isa, re.S | re.M).group(1)
    loads = [m.group(1) for m in re.finditer(r"buffer_load_dword v\d+, v\d+, s\[\d+:\d+\], (\S+) offen", body)]
    assert "buffer_load_dwordx" not in body and len(re.findall("buffer_load", body)) == len(loads)
    # per kind of tile (one operand on the diagonal, else two), eight tokens per operand: three batches first, three inside
    # the run, three that may reach past its end
    assert len(loads) == 9 * 8 * (1 + 2)
    sizes = (8, 16) if next(i for i, o in enumerate(loads) if o != "0") < 3 * 16 else (16, 8)
    pos = 0
    for n in sizes:
        first, inside, past = loads[pos:pos + 3 * n], loads[pos + 3 * n:pos + 6 * n], loads[pos + 6 * n:pos + 9 * n]
        assert all(o == "0" for o in first) and all(o == "0" for o in past)
        assert sum(o != "0" for o in inside) == 3 * (n - n // 8)   # a batch's first token has offset 0
        pos += 9 * n
    assert pos == len(loads)
