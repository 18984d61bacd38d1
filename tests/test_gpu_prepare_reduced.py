"""Points whose coordinates are not canonical: the records and flags of the points that
they stand for, whatever multiple of p is in their 384 bits."""

import numpy as np
import pytest

from oracle.field import P
from paper_2502_11660_amd import api, inputs
from tests import helpers as H

pytestmark = pytest.mark.gpu

MOST = (1 << 384) - 1


@pytest.mark.parametrize("endo", [False, True])
@pytest.mark.parametrize("multiple", [1, 2, 3, 4, 5, 76, MOST])
def test_records_of_the_residues(endo, multiple):
    n = 130
    kw = inputs.nonzero_scalars_mod_r(31, n, stream=1)
    xy, _ = api.gen_points(api.to_device(kw), n)
    rows = H.unsoa(api.to_host(xy), 2, n)
    want, ok = api.points_prepare(xy, n, endo=endo)
    assert int(api.to_host(ok)[0]) == 0
    # every third point's x, y or both
    lift = lambda v: v + min(multiple, (MOST - v) // P) * P  # noqa: E731
    moved = [(lift(x) if i % 3 != 1 else x, lift(y) if i % 3 != 0 else y)
             for i, (x, y) in enumerate(rows)]
    got, status = api.points_prepare(api.to_device(H.soa(moved, 2)), n, endo=endo)
    assert np.array_equal(api.to_host(got), api.to_host(want))
    assert int(api.to_host(status)[0]) == 0
    off = [(x, y) if i != 77 else (x, y - 1 if y > P else y + 1) for i, (x, y) in enumerate(moved)]
    status = api.points_prepare(api.to_device(H.soa(off, 2)), n, endo=endo)[1]
    assert int(api.to_host(status)[0]) & api.MSM_FLAG_OFFCURVE
