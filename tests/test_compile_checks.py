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
