"""Point preparation at the edges of its batching: partial waves, two points
per thread with a partial last turn, and infinity, off-curve and exceptional
points among ordinary ones."""

import numpy as np
import pytest

from oracle import curve, glv, points, te
from oracle.field import P
from paper_2502_11660_amd import api, inputs
from tests import helpers as H

pytestmark = pytest.mark.gpu


def _record(pt):
    return tuple(v * (1 << 384) % P for v in te.to_prepared(te.w_to_te(pt)))


@pytest.mark.parametrize("endo", [False, True])
@pytest.mark.parametrize("n", [1, 63, 65, 257, 131072, 262145])
def test_records(n, endo):
    kw = inputs.nonzero_scalars_mod_r(60 + n, n, stream=1)
    xy, inf = api.gen_points(api.to_device(kw), n)
    rng = np.random.Generator(np.random.PCG64([60, n]))
    sample = sorted({0, n - 1, n // 2, *(int(i) for i in rng.integers(0, n, 12))})
    # other points among them: infinity, the 2-torsion point (-1, 0), off the curve
    odd = [int(i) for i in rng.permutation(n)[:min(3, n - 1)] if int(i) not in (0, n - 1)]
    soa = xy.view(2, 12, n)
    zero_at = api.to_device(np.array(H.int_words(P - 1) + [0] * 12, dtype=np.uint32)).view(2, 12)
    flags = 0
    for kind, i in enumerate(odd):
        if kind == 0:
            inf[i] = 1
        elif kind == 1:
            soa[:, :, i] = zero_at
            flags |= api.MSM_FLAG_EXCEPT
        else:
            soa[0, 0, i] ^= 4
            flags |= api.MSM_FLAG_OFFCURVE
    xyu, status = api.points_prepare(xy, n, inf=inf, endo=endo)
    assert int(api.to_host(status)[0]) == flags
    rec = 2 if endo else 1
    rows = xyu.view(n * rec, 36)
    for i in sample:
        if i in odd:
            continue
        pt = points.fixed_base_mul(inputs.words_to_int(kw[i]))
        assert curve.on_curve(pt)
        for im, q in enumerate([pt, glv.phi(pt)][:rec]):
            got = H.unaos(api.to_host(rows[i * rec + im].contiguous()), 3, 1)[0]
            assert got == _record(q), (i, im)
    if odd:
        got = H.unaos(api.to_host(rows[odd[0] * rec].contiguous()), 3, 1)[0]
        assert got == (0, (1 << 384) % P, 0)


@pytest.mark.parametrize("endo", [False, True])
@pytest.mark.parametrize("n", [131073, 262144, 400001])
def test_records_do_not_depend_on_the_batching(n, endo):
    """Points per thread change with n; a point's record does not."""
    kw = inputs.nonzero_scalars_mod_r(70 + n, n, stream=1)
    xy, inf = api.gen_points(api.to_device(kw), n)
    whole, status = api.points_prepare(xy, n, inf=inf, endo=endo)
    assert int(api.to_host(status)[0]) == 0
    soa = xy.view(2, 12, n)
    rec = 72 if endo else 36
    for lo, hi in ((0, 70000), (n - 50001, n)):
        part, _ = api.points_prepare(soa[:, :, lo:hi].contiguous().reshape(-1), hi - lo,
                                     inf=inf[lo:hi].contiguous(), endo=endo)
        assert bool((part == whole[rec * lo:rec * hi]).all())
