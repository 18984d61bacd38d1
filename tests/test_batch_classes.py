"""Classes of jobs with c = 0: a batch whose jobs plan alone plans whole, however
its default widths coincide or join; a given width keeps a class's limits."""

import pytest

from paper_2502_11660_amd import _lib

S, U, G = _lib.MSM_DIGITS_SIGNED, _lib.MSM_DIGITS_UNSIGNED, _lib.MSM_DIGITS_GLV


def _bytes(sizes, enc, c=0):
    jobs = (_lib.MsmJob * len(sizes))(*[_lib.MsmJob(16, 16, 16, n, c) for n in sizes])
    return _lib.lib().msm_batch_workspace_bytes(jobs, len(sizes), enc)


@pytest.mark.parametrize("enc", [S, U, G])
@pytest.mark.parametrize("sizes", [[1], [7, 7, 7], [1 << 20] * 200, [(1 << 26) - 1] * 4,
                                   [1 << 18] * 600 + [1 << 21] * 60, [1000] * 20000,
                                   list(range(1000, 200000, 997))])
def test_default_widths_plan(sizes, enc):
    total = _bytes(sizes, enc)
    assert total > 0
    # no less than a workspace of the largest job at the narrowest choice
    assert total >= min(_lib.lib().msm_workspace_bytes(max(sizes), c, enc) or total
                        for c in range(4, 21))


@pytest.mark.parametrize("enc", [S, U, G])
def test_a_given_width_keeps_the_limits(enc):
    assert _bytes([1 << 20] * 20, enc, 16) > 0
    assert _bytes([1 << 20] * 300, enc, 16) == 0
    assert _bytes([1 << 20] * 20 + [1 << 26], enc) == 0
