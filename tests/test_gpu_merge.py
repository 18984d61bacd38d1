"""Split buckets of every length around the merge's forms: one to four chunk
partials on one quad, spans of several runs folded in a block, and the first
lengths beyond, many spans to a block and at its last chunk."""

import numpy as np
import pytest

from oracle import msm
from paper_2502_11660_amd import api, inputs

pytestmark = pytest.mark.gpu

UNSIGNED = api.MSM_DIGITS_UNSIGNED


# window 0 holds one bucket of each listed size, in this order; chunks hold 4
# entries here, so a bucket of 4 h + 1 .. 4 h + 4 entries has h heads or so
@pytest.mark.parametrize("sizes", [
    list(range(1, 60)), list(range(60, 1, -1)), [5] * 200, [6, 7, 8] * 40,
    [17, 2, 18, 19, 3, 20, 21] * 8, [4 * h + r for h in (14, 15, 16, 30, 31, 32) for r in (1, 3)],
    [505, 250, 251, 252, 253], [3, 254, 255, 256, 257, 258, 259, 260, 261],
    [500, 12, 500, 13, 500, 30], [4 * h + 2 for h in range(59, 67)]])
@pytest.mark.parametrize("many", [False, True])
def test_bucket_sizes(sizes, many):
    """many: points enough for one-lane chunks; the extra ones have scalar 0."""
    s = np.repeat(np.arange(1, len(sizes) + 1), sizes).tolist()
    n = len(s) + (9000 if many else 0)
    s += [0] * (n - len(s))
    kw = inputs.nonzero_scalars_mod_r(60 + len(sizes), n, stream=1)
    xy, inf = api.gen_points(api.to_device(kw), n)
    xyu, _ = api.points_prepare(xy, n, inf=inf)
    res = api.msm_run(xyu, api.to_device(inputs.ints_to_words(s, 8)), n, 8, UNSIGNED)
    got, flags = api.decode_result(api.to_host(res))
    assert flags == 0
    assert got == msm.closed_form(s, [inputs.words_to_int(r) for r in kw])


@pytest.mark.parametrize("n", [16384, 16385])
@pytest.mark.parametrize("sizes", [list(range(1, 60)), [17, 2, 18, 19, 3, 20, 21] * 8,
                                   [505, 250, 251, 252, 253], [4 * h + 2 for h in range(59, 67)]])
def test_bucket_sizes_on_both_sides_of_the_quad_limit(sizes, n):
    """2^19 digit slots at 32 windows: quads, one point more: lanes."""
    s = np.repeat(np.arange(1, len(sizes) + 1), sizes).tolist()
    s += [0] * (n - len(s))
    kw = inputs.nonzero_scalars_mod_r(60 + len(sizes), n, stream=1)
    xy, inf = api.gen_points(api.to_device(kw), n)
    xyu, _ = api.points_prepare(xy, n, inf=inf)
    res = api.msm_run(xyu, api.to_device(inputs.ints_to_words(s, 8)), n, 8, UNSIGNED)
    got, flags = api.decode_result(api.to_host(res))
    assert flags == 0
    assert got == msm.closed_form(s, [inputs.words_to_int(r) for r in kw])
