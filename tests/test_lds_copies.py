"""The copies from global memory straight into LDS take their LDS address from
M0, and the hardware wants one wait state between a scalar write of M0 and
such a copy.  The compiler does not look for hazards inside assembly strings,
so both the sources and the built library's own code are checked."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2609_32814_amd as P

CSRC = os.path.join(os.path.dirname(P.LIB_PATH), "csrc")
OBJDUMP = shutil.which("llvm-objdump") or "/opt/rocm/llvm/bin/llvm-objdump"


def hazards(lines):
    """Number of copies into LDS, and those right behind a write of M0."""
    copies, bad, after_m0 = 0, [], False
    for line in lines:
        m = re.match(r"\s+([a-z]\w+)(.*)", line.split("//")[0])
        if not m:
            after_m0 = False if line.rstrip().endswith(":") else after_m0
            continue
        op, args = m.groups()
        if re.match(r"(global|buffer|scratch)_load_lds_", op) or (op.startswith("buffer_load") and " lds" in args):
            copies += 1
            if after_m0:
                bad.append(line.strip())
        after_m0 = re.match(r"\s*m0\b", args) is not None
    return copies, bad


def test_hazard_check_sees_one():
    """The check itself, on the oracle's side: two instruction lists."""
    bad = ["\ts_mov_b32 m0, s4\n", "\tglobal_load_lds_dwordx4 v[0:1], off\n"]
    good = [bad[0], "\ts_nop 0\n", bad[1]]
    assert hazards(bad) == (1, ["global_load_lds_dwordx4 v[0:1], off"])
    assert hazards(good) == (1, [])


def test_copies_in_sources_wait_for_m0():
    n = 0
    for f in sorted(os.listdir(CSRC)):
        for s in re.findall(r'asm\s+volatile\(\s*"([^"]*load_lds[^"]*)"', open(os.path.join(CSRC, f)).read()):
            n += 1
            copies, bad = hazards(["\t" + line for line in s.replace(r"\t", "").split(r"\n")])
            assert copies == 1 and not bad, f
    assert n > 0


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="needs llvm-objdump")
def test_copies_in_built_code_wait_for_m0(tmp_path):
    lib = tmp_path / "lib.so"
    shutil.copy(P.LIB_PATH, lib)
    subprocess.run([OBJDUMP, "--offloading", str(lib)], cwd=tmp_path, check=True, capture_output=True)
    total = 0
    for f in sorted(os.listdir(tmp_path)):
        if "gfx950" not in f:
            continue
        out = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", f], cwd=tmp_path, check=True, capture_output=True,
                             text=True).stdout
        copies, bad = hazards(out.splitlines())
        assert not bad, (f, len(bad))
        total += copies
    assert total > 0
