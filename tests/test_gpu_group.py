"""Group aggregation with the affine result in one kernel: every window count
from two up, the identity, results at any 4-byte boundary, many jobs (each one
a field inversion of its own)."""

import numpy as np
import pytest

from oracle import msm
from oracle.field import R_ORDER
from paper_2502_11660_amd import api, inputs

pytestmark = pytest.mark.gpu

SIGNED, UNSIGNED, GLV = api.MSM_DIGITS_SIGNED, api.MSM_DIGITS_UNSIGNED, api.MSM_DIGITS_GLV
EDGES = [0, 1, 2, R_ORDER - 1, R_ORDER - 2, (R_ORDER + 1) // 2, 1 << 251, (1 << 252) % R_ORDER]


@pytest.mark.parametrize("enc", [SIGNED, UNSIGNED, GLV])
@pytest.mark.parametrize("c", [2, 5, 11, 14])
def test_one_point_jobs(c, enc):
    jobs = len(EDGES) + 56
    kw = inputs.nonzero_scalars_mod_r(41, jobs, stream=1)
    sw = inputs.scalars_mod_r(41, jobs, stream=2)
    sw[:len(EDGES)] = inputs.ints_to_words(EDGES, 8)
    xy, inf = api.gen_points(api.to_device(kw), jobs)
    xyu = api.points_prepare(xy, jobs, inf=inf, endo=enc == GLV)[0]
    rec = 36 * (2 if enc == GLV else 1)
    scalars = api.to_device(sw)
    step = api.MSM_RESULT_WORDS + 1  # results at every offset of a 16-byte line
    out = api.words(jobs * step)
    out.fill_(-1)
    slots = [out[j * step:j * step + api.MSM_RESULT_WORDS] for j in range(jobs)]
    b = api.Batch([(xyu[j * rec:(j + 1) * rec], scalars[8 * j:8 * j + 8], slots[j], 1, c)
                   for j in range(jobs)], enc)
    b.run()
    host = api.to_host(out)
    b.destroy()
    for j in range(jobs):
        got, flags = api.decode_result(host[j * step:j * step + api.MSM_RESULT_WORDS])
        assert flags == 0 and got == msm.closed_form_words(sw[j:j + 1], kw[j:j + 1]), j
    between = np.asarray(host)[api.MSM_RESULT_WORDS::step]
    assert (between.astype(np.int64) & 0xffffffff == 0xffffffff).all()
