"""The one-kernel sort at its edges: block sizes, entries per thread, the
largest job and widest buckets it takes and the first beyond, zero digits
kept in place, the status flag, jobs of different sizes in one batch."""

import numpy as np
import pytest

from oracle import msm
from oracle.field import R_ORDER
from paper_2502_11660_amd import api, inputs

pytestmark = pytest.mark.gpu

SIGNED, UNSIGNED, GLV = api.MSM_DIGITS_SIGNED, api.MSM_DIGITS_UNSIGNED, api.MSM_DIGITS_GLV


def _points(n, seed, endo):
    kw = inputs.nonzero_scalars_mod_r(seed, n, stream=1)
    xy, inf = api.gen_points(api.to_device(kw), n)
    return kw, api.points_prepare(xy, n, inf=inf, endo=endo)[0]


def _scalars(n, seed, c):
    """Uniform scalars with runs of zeros, ones, r - 1 and slices at the
    recoding's boundary."""
    sw = inputs.scalars_mod_r(seed, n, stream=2)
    half = sum((1 << (c - 1)) << (c * w) for w in range(253 // c)) % R_ORDER
    special = inputs.ints_to_words([0, 1, R_ORDER - 1, half, half - 1, (1 << 252) % R_ORDER], 8)
    pick = np.random.Generator(np.random.PCG64([seed, 3])).integers(0, 12, n)
    for i in range(6):
        sw[pick == i] = special[i]
    return sw


@pytest.mark.parametrize("enc", [SIGNED, UNSIGNED, GLV])
@pytest.mark.parametrize("n", [1, 255, 1023, 1024, 1025, 4096, 8192, 8193, 16384, 16385])
def test_sizes(n, enc):
    kw, xyu = _points(n, 900 + n, enc == GLV)
    for c in ((5, 9) if n < 8192 else (9,)):
        sw = _scalars(n, 900 + n, c)
        got, flags = api.decode_result(api.to_host(api.msm_run(xyu, api.to_device(sw), n, c, enc)))
        assert flags == 0 and got == msm.closed_form_words(sw, kw), (n, c)


@pytest.mark.parametrize("enc,c", [(UNSIGNED, 13), (UNSIGNED, 14), (SIGNED, 14), (SIGNED, 15),
                                   (GLV, 13), (GLV, 15)])
def test_widest_buckets(enc, c):
    n = 2000
    kw, xyu = _points(n, 77, enc == GLV)
    sw = _scalars(n, 77, c)
    got, flags = api.decode_result(api.to_host(api.msm_run(xyu, api.to_device(sw), n, c, enc)))
    assert flags == 0 and got == msm.closed_form_words(sw, kw)


@pytest.mark.parametrize("enc", [SIGNED, GLV])
def test_range_flag_and_batch_of_sizes(enc):
    """A flagged scalar in one job marks that job alone."""
    sizes = [1, 700, 3000, 40]
    kw, xyu = _points(sum(sizes), 55, enc == GLV)
    sw = inputs.scalars_mod_r(55, sum(sizes), stream=2)
    rec = api.XYU_WORDS * (2 if enc == GLV else 1)
    over = sw.copy()
    over[1 + 650, 7] |= 1 << 29
    s = api.to_device(over)
    res = api.words(api.MSM_RESULT_WORDS * len(sizes)).view(len(sizes), -1)
    jobs, at = [], 0
    for j, n in enumerate(sizes):
        jobs.append((xyu[rec * at:rec * (at + n)], s[8 * at:8 * (at + n)], res[j], n, 7))
        at += n
    b = api.Batch(jobs, enc)
    b.run()
    b.run()
    out = api.to_host(res).reshape(len(sizes), -1)
    at = 0
    for j, n in enumerate(sizes):
        got, flags = api.decode_result(out[j])
        assert flags == (api.MSM_FLAG_RANGE if j == 1 else 0)
        assert got == msm.closed_form_words(sw[at:at + n], kw[at:at + n])
        at += n
    b.destroy()
