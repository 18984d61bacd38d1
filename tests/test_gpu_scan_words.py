"""The sort's scan hands over its blocks' sums as words with a ready bit: workspaces
whose stale words all carry that bit, scans of one block and of many, and fewer
threads in the kernel that clears the words than there are words."""

import pytest

from oracle import msm
from paper_2502_11660_amd import api, inputs

pytestmark = pytest.mark.gpu

SIGNED, UNSIGNED, GLV = api.MSM_DIGITS_SIGNED, api.MSM_DIGITS_UNSIGNED, api.MSM_DIGITS_GLV


@pytest.mark.parametrize("n,c,enc", [(1, 20, UNSIGNED), (3, 20, SIGNED), (17000, 8, SIGNED),
                                     (20000, 14, UNSIGNED), (70000, 16, GLV), (1 << 18, 20, UNSIGNED)])
@pytest.mark.parametrize("stale", [-1, 0, 1 - (1 << 31)])
def test_stale_words(n, c, enc, stale):
    kw = inputs.nonzero_scalars_mod_r(99, n, stream=1)
    xy, inf = api.gen_points(api.to_device(kw), n)
    xyu, _ = api.points_prepare(xy, n, inf=inf, endo=enc == GLV)
    ws = api.workspace(n, c, enc)
    ws.fill_(stale)
    for t in range(2):  # the second on what the first left
        sw = inputs.scalars_mod_r(99 + t, n, stream=2)
        got, flags = api.decode_result(api.to_host(
            api.msm_run(xyu, api.to_device(sw), n, c, enc, ws=ws)))
        assert flags == 0 and got == msm.closed_form_words(sw, kw)
