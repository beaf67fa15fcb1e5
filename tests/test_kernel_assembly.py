"""Properties of the compiled kernels, read from their gfx950 assembly.

Range-checked loads: a buffer load's descriptor bounds its vector and
immediate offset; the scalar offset is left out of that check (LLVM's raw
buffer intrinsics document it so), so a kernel that relies on "past the end
reads zero" must not put a part of its offset there: the scalar offset of every
buffer load is the constant 0.

Registers: the tile loops are laid out to fit the register file; none spills."""
import functools
import os
import re
import subprocess

import pytest

from paper_2609_32831_amd import build

CHECKED = ["select.hip", "attend_decode.hip", "attend_prefill.hip", "score_mfma.hip"]
SOURCES = CHECKED + ["attend_wide.hip", "quantize.hip"]


@functools.lru_cache(None)
def assembly(source):
    if not os.path.exists(build.HIPCC):
        pytest.skip("needs hipcc")
    return subprocess.run([build.HIPCC, *build.FLAGS, "-S", "--cuda-device-only", "-o", "-",
                           os.path.join(build.CSRC, source)], check=True, capture_output=True, text=True).stdout


@pytest.mark.parametrize("source", SOURCES)
def test_no_register_spills(source):
    kernels = re.findall(r"\.name:\s+(\S+).*?\.vgpr_spill_count:\s+(\d+)", assembly(source), re.S)
    assert kernels, "no kernel metadata found"
    assert not [k for k in kernels if k[1] != "0"]


@pytest.mark.parametrize("source", CHECKED)
def test_no_scalar_offset_in_checked_loads(source):
    loads = re.findall(r"^\s*(buffer_load_\w+)\s+([^;\n]*)", assembly(source), re.M)
    assert loads, "no buffer loads found"
    bad = set()
    for op, operands in loads:
        # vdata, vaddr, srsrc, soffset [modifiers]
        fields = re.split(r",\s*(?![^\[]*\])", operands.strip())
        if fields[3].split()[0] != "0":
            bad.add(f"{op} {operands.strip()}")
    assert not bad, sorted(bad)[:5]
