"""The partitioned sort's status flags, counters and many-block path: scalars
out of range anywhere in a batch, digits zero or not beside the flag, one, two
or many large partitions, one or several scan blocks."""

import numpy as np
import pytest

from oracle import msm
from paper_2502_11660_amd import api, inputs

pytestmark = pytest.mark.gpu

SIGNED, UNSIGNED, GLV = api.MSM_DIGITS_SIGNED, api.MSM_DIGITS_UNSIGNED, api.MSM_DIGITS_GLV


def _points(n, seed, endo):
    kw = inputs.nonzero_scalars_mod_r(seed, n, stream=1)
    xy, inf = api.gen_points(api.to_device(kw), n)
    return kw, api.points_prepare(xy, n, inf=inf, endo=endo)[0]


@pytest.mark.parametrize("enc", [SIGNED, UNSIGNED, GLV])
@pytest.mark.parametrize("at", [0, 16384, 19999])
@pytest.mark.parametrize("low", [0, 12345])
def test_flag_in_one_job(enc, at, low):
    """Bits from 253 on are ignored and flag their job alone."""
    n, jobs, c = 20000, 3, 9
    kw, xyu = _points(n, 21, enc == GLV)
    rec = 36 * (2 if enc == GLV else 1)
    batch, words = [], []
    for j in range(jobs):
        sw = inputs.scalars_mod_r(31 + j, n, stream=2)
        if j == 1:
            sw[at] = inputs.ints_to_words([low], 8)[0]
        words.append(sw.copy())
        if j == 1:
            sw[at, 7] |= np.uint32(1 << 31 | 1 << 29)
        batch.append((xyu[:rec * n], api.to_device(sw), api.words(api.MSM_RESULT_WORDS), n, c))
    b = api.Batch(batch, enc)
    for _ in range(2):
        b.run()
        for j in range(jobs):
            got, flags = api.decode_result(api.to_host(batch[j][2]))
            assert flags == (api.MSM_FLAG_RANGE if j == 1 else 0), j
            assert got == msm.closed_form_words(words[j], kw), j
    b.destroy()


# distinct scalars; c; points: partitions beyond the LDS stage in one window, in
# all, in every partition of a window, many items each
@pytest.mark.parametrize("enc", [SIGNED, UNSIGNED, GLV])
@pytest.mark.parametrize("n,distinct,c", [(16385, 16385, 7), (30000, 1, 12), (70001, 2, 13),
                                          (70001, 300, 16), (150000, 5, 10)])
def test_few_distinct_scalars(enc, n, distinct, c):
    kw, xyu = _points(n, 5, enc == GLV)
    sw = inputs.scalars_mod_r(9, distinct, stream=2)[np.arange(n) * 7 % distinct]
    got, flags = api.decode_result(api.to_host(api.msm_run(xyu, api.to_device(sw), n, c, enc)))
    assert flags == 0 and got == msm.closed_form_words(sw, kw)
