"""Range-checked loads: a buffer load's descriptor bounds its vector and
immediate offset; the scalar offset is left out of that check (LLVM's raw
buffer intrinsics document it so), so a kernel that relies on "past the end
reads zero" must not put a part of its offset there.  Checked on the gfx950
assembly of every kernel source: the scalar offset of every buffer load is the
constant 0."""
import os
import re
import subprocess

import pytest

from paper_2609_32831_amd import build

SOURCES = ["select.hip", "attend_decode.hip", "attend_prefill.hip", "score_mfma.hip"]


@pytest.mark.parametrize("source", SOURCES)
def test_no_scalar_offset_in_checked_loads(source, tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("needs hipcc")
    out = tmp_path / "kernels.s"
    subprocess.run([build.HIPCC, *build.FLAGS, "-S", "--cuda-device-only", "-o", str(out),
                    os.path.join(build.CSRC, source)], check=True, capture_output=True)
    loads = re.findall(r"^\s*(buffer_load_\w+)\s+([^;\n]*)", out.read_text(), re.M)
    assert loads, "no buffer loads found"
    bad = set()
    for op, operands in loads:
        # vdata, vaddr, srsrc, soffset [modifiers]
        fields = re.split(r",\s*(?![^\[]*\])", operands.strip())
        if fields[3].split()[0] != "0":
            bad.add(f"{op} {operands.strip()}")
    assert not bad, sorted(bad)[:5]
