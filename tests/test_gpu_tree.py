"""The aggregation tree's forms by bucket bits and schedule: the fused first two
levels, lane levels, quad levels one and two at a time, the window's last
levels in one block, up to the widest windows."""

import pytest

from oracle import msm
from paper_2502_11660_amd import api, inputs

pytestmark = pytest.mark.gpu

SIGNED, UNSIGNED, GLV = api.MSM_DIGITS_SIGNED, api.MSM_DIGITS_UNSIGNED, api.MSM_DIGITS_GLV


def _inputs(n, endo):
    kw = inputs.nonzero_scalars_mod_r(300 + n, n, stream=1)
    sw = inputs.scalars_mod_r(300 + n, n, stream=2)
    xy, inf = api.gen_points(api.to_device(kw), n)
    return kw, sw, api.points_prepare(xy, n, inf=inf, endo=endo)[0]


@pytest.mark.parametrize("enc,c", [(SIGNED, 18), (SIGNED, 20), (UNSIGNED, 20), (GLV, 20)])
def test_widest_windows(enc, c):
    n = 600
    kw, sw, xyu = _inputs(n, enc == GLV)
    got, flags = api.decode_result(api.to_host(api.msm_run(xyu, api.to_device(sw), n, c, enc)))
    assert flags == 0 and got == msm.closed_form_words(sw, kw)


# bucket bits 1 .. 11 of four or more windows, lanes from the first level on
# (tree_quad 1), quads only, and the one-block levels from 1, 40 or 500 outputs
# over all windows
@pytest.mark.parametrize("c", [2, 3, 4, 5, 8, 9, 10, 12])
@pytest.mark.parametrize("sched", [{"tree_quad": 1}, {"tree_quad": 1 << 20}, {"tree_wide": 1},
                                   {"tree_quad": 1, "tree_wide": 40},
                                   {"tree_quad": 1 << 20, "tree_wide": 500}])
def test_schedules_by_bucket_bits(c, sched):
    n = 90
    kw, sw, xyu = _inputs(n, False)
    want = msm.closed_form_words(sw, kw)
    for enc in (SIGNED, UNSIGNED):
        res = api.words(api.MSM_RESULT_WORDS)
        b = api.Batch([(xyu, api.to_device(sw), res, n, c, sched)], enc)
        b.run()
        got, flags = api.decode_result(api.to_host(res))
        b.destroy()
        assert flags == 0 and got == want, enc
