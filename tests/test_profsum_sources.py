"""The sources whose hash says whether recorded counters still describe a kernel:
its unit and every device header that the unit includes."""

import re
import shutil

from paper_2502_11660_amd import profsum

CSRC = profsum.CSRC


def test_accumulation_sources_are_complete():
    assert {CSRC + n for n in ("k_accum.hip", "mad64.hpp", "fe29.hpp", "curve29.hpp", "curve.hpp",
                               "field.hpp", "common.hpp", "quad29.hpp")} <= set(profsum.ACCUM_SOURCES)


def test_sort_sources_are_complete():
    got = profsum.with_headers([CSRC + "k_sort.hip"])
    assert got[0] == CSRC + "k_sort.hip" and len(got) == len(set(got))
    assert {CSRC + n for n in ("common.hpp", "convert.hpp", "small_sort.hpp")} <= set(got)


def test_a_change_of_any_header_changes_the_hash(tmp_path, monkeypatch):
    for p in profsum.ACCUM_SOURCES:
        dst = tmp_path / p
        dst.parent.mkdir(parents=True, exist_ok=True)
        shutil.copy(profsum.ROOT + "/" + p, dst)
        assert re.match(r"paper_2502_11660_amd/csrc/\w+\.(hip|hpp)$", p)
    monkeypatch.setattr(profsum, "ROOT", str(tmp_path))
    before = profsum.sources_sha256(profsum.ACCUM_SOURCES)
    (tmp_path / (CSRC + "mad64.hpp")).write_text("changed")
    assert profsum.sources_sha256(profsum.ACCUM_SOURCES) != before
