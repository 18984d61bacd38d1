"""Bucket spans at the edges of the accumulation's and the merges' forms: one
quad or one lane per chunk, sums of a few chunk partials on one quad, segments
of longer spans on many blocks, and more segments than a block has quads."""

import pytest

from oracle import msm
from paper_2502_11660_amd import api, inputs

pytestmark = pytest.mark.gpu

UNSIGNED = api.MSM_DIGITS_UNSIGNED
# chunks hold 4 entries here: the first bucket's n - 5 entries span
# ceil / 4 of them.  Up to 8192 points (2^18 digit slots at 32 windows) run on
# quads, more on lanes; spans of 8 and 9 chunks, of 128 and 129 heads (one
# and two segments), of more than 64 segments.
SIZES = [6, 9, 10, 37, 38, 41, 42, 516, 517, 521, 8192, 8193, 40000]


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("first", [0, 5])
def test_one_long_bucket(n, first):
    """Scalars 1 (the first `first` points) and 2: window 0 holds two buckets,
    the other windows nothing."""
    kw = inputs.nonzero_scalars_mod_r(700 + n, n, stream=first)
    xy, inf = api.gen_points(api.to_device(kw), n)
    xyu, _ = api.points_prepare(xy, n, inf=inf)
    s = [1] * first + [2] * (n - first)
    res = api.msm_run(xyu, api.to_device(inputs.ints_to_words(s, 8)), n, 8, UNSIGNED)
    got, flags = api.decode_result(api.to_host(res))
    assert flags == 0
    assert got == msm.closed_form(s, [inputs.words_to_int(r) for r in kw])


@pytest.mark.parametrize("n", [8192, 8193])
def test_uniform_digits_on_both_sides_of_the_quad_limit(n):
    kw = inputs.nonzero_scalars_mod_r(800 + n, n, stream=1)
    sw = inputs.scalars_mod_r(800 + n, n, stream=2)
    xy, inf = api.gen_points(api.to_device(kw), n)
    xyu, _ = api.points_prepare(xy, n, inf=inf)
    res = api.msm_run(xyu, api.to_device(sw), n, 8, UNSIGNED)
    got, flags = api.decode_result(api.to_host(res))
    assert flags == 0 and got == msm.closed_form_words(sw, kw)
