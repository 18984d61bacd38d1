"""The columns of multiply-adds of the signed 29-bit core (mad64.hpp) are inline
asm blocks whose carry-outs are early-clobber outputs: no multiply-add of a
block reads a scalar register that an earlier one of the block wrote, in any
translation unit that uses the core."""

import concurrent.futures as cf
import os
import re
import shutil
import subprocess

import pytest

from paper_2502_11660_amd import build as B

UNITS = ["k_accum.hip", "k_agg.hip", "k_chain.hip", "k_elementwise.hip", "k_segment.hip"]
MAD = re.compile(r"v_mad_(?:i64_i32|u64_u32) v\[\d+:\d+\], s\[(\d+):(\d+)\], (\S+?), (\S+?), (.+)")


def hazards(text):
    found = []
    for block in re.findall(r"ASMSTART(.*?)ASMEND", text, re.S):
        written = set()
        for line in block.split("\n"):
            m = MAD.match(line.strip())
            if not m:
                continue
            read = set()
            for op in m.group(3, 4, 5):
                r = re.match(r"s(?:(\d+)$|\[(\d+):(\d+)\])", op)
                if r:
                    read |= {int(x) for x in r.groups() if x}
            if read & written:
                found.append(line.strip())
            written |= {int(m.group(1)), int(m.group(2))}
    return found


def test_scanner_catches_a_planted_overlap():
    bad = "\n".join([";;#ASMSTART", "v_mad_i64_i32 v[70:71], s[10:11], v107, s7, v[70:71]",
                     "v_mad_i64_i32 v[70:71], s[10:11], v111, s11, v[70:71]", ";;#ASMEND"])
    assert len(hazards(bad)) == 1
    assert hazards(bad.replace("s11, v[70:71]", "s12, v[70:71]")) == []


@pytest.mark.skipif(shutil.which(B.hipcc()) is None and not os.path.exists(B.hipcc()),
                    reason="hipcc not available")
def test_no_carry_out_overlaps_an_sgpr_factor(tmp_path):
    inc = ["-I", os.path.join(B.ROOT, "include"), "-I", B.CSRC]

    def asm_of(unit):
        out = tmp_path / (unit + ".s")
        subprocess.run([B.hipcc(), *B.HIPCC_FLAGS, *inc, "--cuda-device-only", "-S", "-o", str(out),
                        os.path.join(B.CSRC, unit)], check=True, capture_output=True)
        return unit, out.read_text()

    with cf.ThreadPoolExecutor(len(UNITS)) as ex:
        for unit, text in ex.map(asm_of, UNITS):
            blocks = re.findall(r"ASMSTART(.*?)ASMEND", text, re.S)
            assert sum("v_mad_i64_i32" in b for b in blocks) > 100, unit
            assert hazards(text) == [], unit
