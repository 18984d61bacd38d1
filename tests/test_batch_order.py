"""Whether a batch plans, and what it needs, does not depend on the order of jobs
with c = 0 and jobs with a given width."""

import random

import pytest

from paper_2502_11660_amd import _lib

S, U, G = _lib.MSM_DIGITS_SIGNED, _lib.MSM_DIGITS_UNSIGNED, _lib.MSM_DIGITS_GLV


def _bytes(jobs, enc):
    arr = (_lib.MsmJob * len(jobs))(*[_lib.MsmJob(16, 16, 16, n, c) for n, c in jobs])
    return _lib.lib().msm_batch_workspace_bytes(arr, len(jobs), enc)


@pytest.mark.parametrize("enc,c", [(G, 16), (S, 16), (U, 16), (S, 20)])
def test_default_jobs_leave_room_for_a_given_width(enc, c):
    """Each part plans alone; together they are more than a class holds."""
    loose, given = [(1 << 20, 0)] * 60, [(1 << 20, c)] * (70 if c == 16 else 100)
    assert _bytes(loose, enc) > 0 and _bytes(given, enc) > 0
    total = _bytes(given + loose, enc)
    assert total > 0
    assert _bytes(loose + given, enc) == total
    mixed = loose + given
    random.Random(c).shuffle(mixed)
    assert _bytes(mixed, enc) == total
