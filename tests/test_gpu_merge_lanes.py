"""Split buckets of lanes: jobs of more than 2^19 digit slots whose zero digits the
partitioned sort drops, so that the few entries are cut into chunks of four; uniform
digits on both sides of the quads' limit; and a sort whose last group of tiles is a
partial one, with groups of sixteen."""

import numpy as np
import pytest

from oracle import msm
from paper_2502_11660_amd import api, inputs

pytestmark = pytest.mark.gpu

UNSIGNED, SIGNED = api.MSM_DIGITS_UNSIGNED, api.MSM_DIGITS_SIGNED


def _check(n, c, enc, scalars, seed):
    kw = inputs.nonzero_scalars_mod_r(seed, n, stream=1)
    xy, inf = api.gen_points(api.to_device(kw), n)
    xyu, _ = api.points_prepare(xy, n, inf=inf)
    got, flags = api.decode_result(api.to_host(api.msm_run(xyu, api.to_device(scalars), n, c, enc)))
    assert flags == 0 and got == msm.closed_form_words(scalars, kw)


# window 0 holds one bucket of each size, in this order; a bucket of 4 h + 1 ..
# 4 h + 4 entries has h heads or so.  63 heads are summed by one block, 64 and more
# by segments of 128
@pytest.mark.parametrize("sizes", [
    list(range(1, 60)), list(range(60, 1, -1)), [5] * 200, [6, 7, 8] * 40,
    [17, 2, 18, 19, 3, 20, 21] * 8, [4 * h + r for h in (14, 15, 16, 30, 31, 32) for r in (1, 3)],
    [505, 250, 251, 252, 253], [3, 254, 255, 256, 257, 258, 259, 260, 261],
    [500, 12, 500, 13, 500, 30], [4 * h + 2 for h in range(59, 67)],
    [511, 512, 513, 514, 516, 517, 521, 1100], [40000]])
def test_bucket_sizes(sizes):
    s = np.repeat(np.arange(1, len(sizes) + 1), sizes)
    n = max(16385, s.size) + 100  # 32 windows: more than 2^19 digit slots
    sw = np.zeros((n, 8), dtype=np.uint32)
    sw[50:50 + s.size, 0] = s
    _check(n, 8, UNSIGNED, sw, 61)


@pytest.mark.parametrize("n", [16384, 16385])
def test_uniform_digits_on_both_sides_of_the_quad_limit(n):
    _check(n, 8, UNSIGNED, inputs.scalars_mod_r(62, n, stream=2), 62)


def test_partial_group_of_sixteen_tiles():
    """20 bits: 2^11 partitions a window and groups of 16 tiles of 8192 digits, the
    last group of a window with 777."""
    n = (1 << 21) + 777
    rng = np.random.default_rng(63)
    sw = rng.integers(0, 1 << 32, size=(n, 8), dtype=np.uint32)
    sw[:, 7] &= 0x0FFFFFFF
    _check(n, 20, SIGNED, sw, 63)
