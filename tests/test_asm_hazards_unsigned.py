"""The unsigned columns of multiply-adds (fe28.hpp's, mad64.hpp) are compiled into
k_fieldvar.hip alone: there, as in the signed ones, no multiply-add of an asm block
reads a scalar register that an earlier one of the block wrote as its carry-out."""

import os
import re
import shutil
import subprocess

import pytest

from paper_2502_11660_amd import build as B
from tests.test_asm_hazards_signed import hazards

FACTOR = re.compile(r"v_mad_u64_u32 v\[\d+:\d+\], s\[\d+:\d+\], v\d+, s\d+,")


def test_scanner_catches_a_planted_overlap():
    bad = "\n".join([";;#ASMSTART", "v_mad_u64_u32 v[70:71], s[10:11], v107, s7, v[70:71]",
                     "v_mad_u64_u32 v[70:71], s[10:11], v111, s11, v[70:71]", ";;#ASMEND"])
    assert len(hazards(bad)) == 1
    assert hazards(bad.replace("s11, v[70:71]", "s12, v[70:71]")) == []


@pytest.mark.skipif(shutil.which(B.hipcc()) is None and not os.path.exists(B.hipcc()),
                    reason="hipcc not available")
def test_no_carry_out_overlaps_an_sgpr_factor(tmp_path):
    out = tmp_path / "k_fieldvar.s"
    subprocess.run([B.hipcc(), *B.HIPCC_FLAGS, "-I", os.path.join(B.ROOT, "include"), "-I", B.CSRC,
                    "--cuda-device-only", "-S", "-o", str(out),
                    os.path.join(B.CSRC, "k_fieldvar.hip")], check=True, capture_output=True)
    text = out.read_text()
    blocks = re.findall(r"ASMSTART(.*?)ASMEND", text, re.S)
    # the blocks with a factor in a scalar register, most of them of several products
    with_factor = [b for b in blocks if FACTOR.search(b)]
    assert len(with_factor) >= 20
    assert sum(b.count("v_mad_u64_u32") > 1 for b in with_factor) >= 20
    assert hazards(text) == []
