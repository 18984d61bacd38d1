"""The width that c = 0 picks: narrower ones where a scratch is too small for
the best, workspaces sized for msm_default_window with unsigned digits, batches
whose jobs join widths, single MSMs around the changes of width."""

import pytest

from oracle import msm
from paper_2502_11660_amd import _lib, api, inputs

pytestmark = pytest.mark.gpu

SIGNED, UNSIGNED, GLV = api.MSM_DIGITS_SIGNED, api.MSM_DIGITS_UNSIGNED, api.MSM_DIGITS_GLV


def _points(n, seed, endo):
    kw = inputs.nonzero_scalars_mod_r(seed, n, stream=1)
    xy, inf = api.gen_points(api.to_device(kw), n)
    return kw, api.points_prepare(xy, n, inf=inf, endo=endo)[0]


@pytest.mark.parametrize("enc", [SIGNED, UNSIGNED, GLV])
@pytest.mark.parametrize("n", [1, 64, 300, 3000, 15000, 60000])
def test_single(enc, n):
    kw, xyu = _points(n, 70 + n, enc == GLV)
    sw = inputs.scalars_mod_r(70 + n, n, stream=2)
    got, flags = api.decode_result(api.to_host(api.msm_run(xyu, api.to_device(sw), n, 0, enc)))
    assert flags == 0 and got == msm.closed_form_words(sw, kw)


def test_noalloc_takes_a_width_that_fits():
    n = 180000
    assert api.workspace_bytes(n, 0, GLV) > _lib.MSM_NOALLOC_SCRATCH_BYTES
    assert api.workspace_bytes(n, 13, GLV) <= _lib.MSM_NOALLOC_SCRATCH_BYTES
    kw, xyu = _points(n, 3, True)
    sw = inputs.scalars_mod_r(3, n, stream=2)
    got, flags = api.decode_result(api.to_host(api.msm_run_noalloc(xyu, api.to_device(sw), n, 0, GLV)))
    assert flags == 0 and got == msm.closed_form_words(sw, kw)


@pytest.mark.parametrize("n", [300, 20000, 90000])
def test_unsigned_in_a_workspace_of_the_default_window(n):
    kw, xyu = _points(n, 4, False)
    sw = inputs.scalars_mod_r(4, n, stream=2)
    ws = api.workspace(n, api.default_window(n), UNSIGNED)
    got, flags = api.decode_result(api.to_host(api.msm_run(xyu, api.to_device(sw), n, 0, UNSIGNED, ws=ws)))
    assert flags == 0 and got == msm.closed_form_words(sw, kw)


@pytest.mark.parametrize("enc", [SIGNED, UNSIGNED, GLV])
@pytest.mark.parametrize("sizes", [[5], [64, 90, 125, 70], [300, 5000, 40000, 9000, 700, 33000],
                                   [20000, 1, 17000, 14000, 3]])
def test_batch(enc, sizes):
    kw, xyu = _points(max(sizes), 8, enc == GLV)
    rec = 36 * (2 if enc == GLV else 1)
    jobs, words = [], []
    for j, n in enumerate(sizes):
        sw = inputs.scalars_mod_r(80 + j, n, stream=2)
        words.append(sw)
        jobs.append((xyu[:rec * n], api.to_device(sw), api.words(api.MSM_RESULT_WORDS), n,
                     9 if j == 3 else 0))
    b = api.Batch(jobs, enc)
    b.run()
    for j, n in enumerate(sizes):
        got, flags = api.decode_result(api.to_host(jobs[j][2]))
        assert flags == 0 and got == msm.closed_form_words(words[j], kw[:n]), j
    b.destroy()
