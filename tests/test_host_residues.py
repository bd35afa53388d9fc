"""The arithmetic of the products by residues (csrc/residue_math.hpp: moduli and tables, an entry's and a sum's residue, the value that
residues stand for, scales) is shared by kernels and host.  tests/residue_check.cpp runs it against 128-bit integers, with UBSan."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2603_28845_amd", "csrc")


@pytest.mark.parametrize("flags", [["-O2"], ["-O1", "-g", "-fsanitize=undefined", "-fno-sanitize-recover=all"]])
def test_residue_arithmetic(tmp_path, flags):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no C++ compiler")
    exe = tmp_path / "residue_check"
    cmd = [gxx, "-std=c++17", "-Wall", "-Wextra", "-Werror", *flags, os.path.join(HERE, "residue_check.cpp"), "-o", str(exe)]
    b = subprocess.run(cmd, capture_output=True, text=True)
    if len(flags) > 1 and "ubsan" in b.stderr:
        pytest.skip("sanitizer runtime not available to this compiler")
    assert b.returncode == 0, b.stderr
    env = dict(os.environ)
    env.pop("LD_PRELOAD", None)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=600, env=env)
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.split()[0] == "ok" and int(r.stdout.split()[1]) > 20000000


@pytest.mark.parametrize("old,new", [
    ("256, 251,", "256, 255,"),                                  # 3 divides 249 too
    ("ENTRY_N2 = 346000", "ENTRY_N2 = 1 << 19"),                 # an entry's residue would leave 8 bits
    ("MAX_K = 1 << 15", "MAX_K = 1 << 16"),                      # the accumulators' start and the quotients
    ("BOUND_EXP = 109", "BOUND_EXP = 111"),                      # longer entries
])
def test_residue_margins_are_asserted(tmp_path, old, new):
    """Moduli, bound and inner range cannot be changed past what the 8-bit residues and 32-bit sums hold."""
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no C++ compiler")
    with open(os.path.join(CSRC, "residue_math.hpp")) as f:
        text = f.read()
    assert text.count(old) == 1
    src = tmp_path / "m.cpp"
    src.write_text(text.replace(old, new))
    r = subprocess.run([gxx, "-std=c++17", "-fsyntax-only", str(src)], capture_output=True, text=True)
    assert r.returncode != 0 and "static assertion failed" in r.stderr
