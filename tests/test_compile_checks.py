"""What the device headers promise at compile time."""

import os
import shutil
import subprocess

import pytest

from paper_2502_11660_amd import build as B

pytestmark = pytest.mark.skipif(shutil.which(B.hipcc()) is None and not os.path.exists(B.hipcc()),
                                reason="hipcc not available")


def _compiles(tmp_path, text):
    src = tmp_path / "unit.hip"
    src.write_text(text)
    return subprocess.run([B.hipcc(), *B.HIPCC_FLAGS, "-I", os.path.join(B.ROOT, "include"), "-I",
                           B.CSRC, "--cuda-device-only", "-fsyntax-only", str(src)],
                          capture_output=True, text=True)


def test_constant_read_as_a_record_is_aligned_like_one(tmp_path):
    r = _compiles(tmp_path, '#include "quad29.hpp"\n'
                            'static_assert(__alignof__(msm::kTwoR) >= 16, "16-byte loads");\n')
    assert r.returncode == 0, r.stderr


@pytest.mark.parametrize("args,ok", [("true, 12, 12", True), ("true, 13, 12", True),
                                     ("false, 14, 0", True), ("false, 0, 14", True),
                                     ("true, 1, 3", False), ("true, 12, 13", False),
                                     ("true, 15, 0", False), ("true, 0, 0", False),
                                     ("false, 2, 2", False)])
def test_columns_without_a_block_do_not_compile(tmp_path, args, ok):
    """mad64_block: a number of products with no asm block would add nothing."""
    sign = args.startswith("true")
    acc, word = ("int64_t", "int32_t") if sign else ("uint64_t", "uint32_t")
    r = _compiles(tmp_path, '#include "mad64.hpp"\n__global__ void k(%s* a, const %s* x) {\n'
                            '  %s acc = *a;\n  msm::mad64_block<%s>(acc, x, x, x, x);\n'
                            '  *a = acc;\n}\n' % (acc, word, acc, args))
    assert (r.returncode == 0) == ok, r.stderr
