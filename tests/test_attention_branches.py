"""Matrix instructions ignore EXEC, so a wave that skips a key tile has to jump over them: in the assembly
of the attention kernels, whatever narrows EXEC is followed by a jump for the case that no lane is
left before the next matrix instruction."""
import os
import re
import subprocess

import pytest

from paper_2502_00425_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
NARROWS = re.compile(r"s_\w*saveexec\w* |s_(?:and|andn2|mov|xor|cselect)_b64 exec\b")
JUMPS = re.compile(r"s_cbranch_exec(?:z|nz) ")
WIDENS = re.compile(r"s_or_b64 exec, exec|s_mov_b64 exec, -1")


def unguarded(lines):
    """Line numbers of matrix instructions that run on whatever a narrowed EXEC has left."""
    bad, open_ = [], False
    for i, line in enumerate(lines):
        if WIDENS.search(line) or JUMPS.search(line):
            open_ = False
        elif NARROWS.search(line):
            open_ = True
        elif "v_mfma" in line and open_:
            bad.append(i)
    return bad


def test_the_check_sees_a_missing_jump():
    jump = ["s_and_saveexec_b64 s[2:3], vcc", "s_cbranch_execz .L1", "v_mfma_f32_32x32x16_f16 a", "s_or_b64 exec, exec, s[2:3]"]
    assert unguarded(jump) == [] and unguarded([jump[0], *jump[2:]]) == [1]


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_skipped_tiles_are_jumped_over(tmp_path):
    out = tmp_path / "attention.s"
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([HIPCC, *flags, "-S", "--cuda-device-only", "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC,
                    os.path.join(build.CSRC, "attention.hip"), "-o", str(out)], check=True, capture_output=True)
    bodies = re.findall(r"^(\S*aifs_attention_kernel\S*):[^\n]*\n(.*?)\n\.Lfunc_end", out.read_text(), re.S | re.M)
    assert len(bodies) == 3
    for name, body in bodies:
        lines = [l.strip() for l in body.split("\n")]
        assert sum("v_mfma" in l for l in lines) >= 64, name
        assert unguarded(lines) == [], name
